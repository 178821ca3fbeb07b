"""The depth order inside the tile lists against the oracle's sorted instance list, bit-exact, where
the depth sort changes its way: candidate counts around the one-workgroup sort's keys per thread
and its end, candidates that are not rendered, equal depths, and depths on both sides of 8192 (three
passes or four), in frames that follow each other on one context."""
import numpy as np
import pytest

import oracle
from paper_2408_12894_amd import synth
from parity import check_instances, check_keys

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FACTORS = {"near": (1.0, 1.0), "across": (0.5, 4000.0), "far": (3000.0, 2e6)}


def _renderer():
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return render.Renderer(0)


def _scene(n, depths, seed=91):
    """Specks in front of the camera and behind it, each moved along its line of sight; every
    third one at the depth of the one before."""
    rng = np.random.default_rng(seed)
    sc = synth.uniform_scene(n, seed=seed, s_mu=-5.0, s_sigma=0.3, extent=1.5)
    eye = np.array((0.0, 0.0, -3.0))
    lo, hi = FACTORS[depths]
    f = np.exp(rng.uniform(np.log(lo), np.log(hi), n)) if hi > lo else np.ones(n)
    p = sc.means.astype(np.float64) - eye
    p[2::3] = p[1::3][: len(p[2::3])] * (1.0, -1.0, 1.0)
    f[2::3] = f[1::3][: len(f[2::3])]
    p[::7, 2] *= -1.0
    sc.means[:] = (eye + p * f[:, None]).astype(np.float32)
    sc.log_scales += np.log(f).astype(np.float32)[:, None]
    return sc


def _check(r, n, depths):
    from paper_2408_12894_amd import render
    print(f"[case] depth sort n={n} {depths}", flush=True)
    scene = _scene(n, depths)
    cam = synth.look_at_camera((0.0, 0.0, -3.0), (0, 0, 0), 200, 152)
    r.render_level(render.GaussianLevel.from_scene(scene), cam)
    torch.cuda.synchronize()
    view = r.view()
    k = oracle.keys(*scene.arrays()[:4], scene.s_min, cam)
    check_keys(view, k)
    check_instances(view, k)
    vis = k["visible"].astype(bool)
    far = vis & (k["depth_bits"] >= np.float32(8192.0).view(np.uint32))
    assert far.any() == (depths != "near") and (n < 64 or not vis.all())


@pytest.mark.parametrize("depths", ["near", "across"])
@pytest.mark.parametrize("n", [2048, 2049, 4096, 4097, 8192, 8193])
def test_order_around_the_ways(n, depths):
    _check(_renderer(), n, depths)


def test_one_candidate():
    _check(_renderer(), 1, "near")


def test_far_and_near_frames_in_turn():
    r = _renderer()
    for n, depths in ((9000, "near"), (9000, "far"), (12_000, "across"), (9000, "near"), (3000, "far"), (20_000, "far")):
        _check(r, n, depths)
