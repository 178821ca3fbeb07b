"""Overlap pruning where points have few neighbours, against the brute-force oracle: sets that a thread
per point settles (32,768 points or more, at most one in 256 with more than 320 in the buckets around it),
sets just outside that, points of such a set that waves take beside it, and the sizes around 256 points, whose
keys hold no subcells. Decisions and distances are the same FP64 operations on both sides: compared
bit for bit."""
import numpy as np
import pytest

from test_gpu_prune_levels import D_OP, _check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CELL = 3 * D_OP * 1.001


def _uniform(n, gap, seed=7):
    return np.random.default_rng(seed).uniform(-0.5, 0.5, (n, 3)) * gap * D_OP * n ** (1 / 3)


@pytest.mark.parametrize("n", [32_767, 32_768, 33_001])
@pytest.mark.parametrize("gap", [0.9, 1.6, 2.0, 3.0, 10.0])
def test_uniform_sets(n, gap):
    print(f"[case] {n} points {gap} d_op apart", flush=True)
    _check(_uniform(n, gap).astype(np.float32))


@pytest.mark.parametrize("per_cell,blocks", [(13, 1), (13, 12), (40, 3)])
def test_crowded_points_in_a_sparse_set(per_cell, blocks):
    """Blocks of 3 x 3 x 3 cells: only their middle cells' points have all of a block around them. 13 and
    156 such points (n / 256 is 132), and blocks crowded throughout."""
    print(f"[case] {blocks} blocks of {per_cell} points per cell", flush=True)
    rng = np.random.default_rng(blocks)
    cells = np.stack(np.meshgrid(range(3), range(3), range(3), indexing="ij"), -1).reshape(-1, 1, 3)
    parts = [_uniform(33_000, 4.0)]
    for b in range(blocks):
        at = np.floor(rng.uniform(-20, 20, 3))
        parts.append(((at + cells + rng.random((27, per_cell, 3))) * CELL).reshape(-1, 3))
    m = np.concatenate(parts).astype(np.float32)
    _check(m[rng.permutation(m.shape[0])])


def test_equal_points_in_a_sparse_set():
    print("[case] pairs to sixes of equal points", flush=True)
    m = _uniform(36_000, 3.0)
    for k, first in ((2, 0), (3, 6000), (4, 12_000), (6, 18_000)):
        m[first:first + 600 * k] = np.repeat(m[first:first + 600], k, axis=0)
    _check(m.astype(np.float32))


@pytest.mark.parametrize("n", [4, 255, 256, 257, 512])
def test_small_sets(n):
    print(f"[case] {n} points", flush=True)
    for gap in (0.2, 0.9, 2.0):
        _check(_uniform(n, gap, seed=n).astype(np.float32))
