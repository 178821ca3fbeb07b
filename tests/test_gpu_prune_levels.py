"""Overlap pruning's subcell search against the brute-force oracle: cells whose occupancy lies
around the thresholds of its three levels, cores much denser than their halo (searches that start
fine and end in the whole cells), coordinates around zero and far from it, and equal points.
Decisions and distances are the same FP64 operations on both sides: compared bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2408_12894_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

D_OP = 0.1


def _check(means):
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sc = synth.uniform_scene(means.shape[0], seed=1)
    lv = render.GaussianLevel.from_arrays(means, *sc.arrays()[1:], s_min=2 * D_OP)
    keep, n_keep, davg = render.Renderer(0).overlap_prune(lv, D_OP, with_d_avg=True)
    keep, davg = keep.cpu().numpy(), davg.cpu().numpy()
    ok, od = oracle.overlap_prune(means, D_OP)
    np.testing.assert_array_equal(keep, ok)
    found = np.isfinite(davg)
    np.testing.assert_array_equal(davg[found], od[found])
    assert np.all(od[~found] >= D_OP)
    assert n_keep == int(keep.sum())


@pytest.mark.parametrize("count", [11, 12, 95, 96, 767, 768, 769])
@pytest.mark.parametrize("offset", [0.0, -37.3])
def test_cells_around_the_thresholds(count, offset):
    """`count` points per cell of edge 3 d_op over a 3 x 3 x 2 block of cells."""
    print(f"[case] {count} points per cell, offset {offset}", flush=True)
    rng = np.random.default_rng(count)
    cells = np.stack(np.meshgrid(range(3), range(3), range(2), indexing="ij"), -1).reshape(-1, 1, 3)
    m = (cells + rng.random((18, count, 3))) * 3 * D_OP + offset
    _check(m.reshape(-1, 3).astype(np.float32))


@pytest.mark.parametrize("core", [0.002, 0.02, 0.08])
def test_dense_core_in_a_sparse_halo(core):
    print(f"[case] core of width {core}", flush=True)
    rng = np.random.default_rng(5)
    m = np.concatenate([rng.normal(0, core, (2500, 3)), rng.normal(0, 0.6, (1500, 3)), rng.normal(0, 3.0, (800, 3)),
                        np.repeat(rng.normal(0, 0.3, (40, 3)), 5, axis=0)]).astype(np.float32)
    _check(m[rng.permutation(m.shape[0])])
