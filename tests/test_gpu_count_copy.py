"""Counts read back by a copy, for where coherent host memory is not to be had (forced by
FLOD_COUNT_COPY=1 when the context is made), beside counts that the kernels write to the host: the same
calls on a context of each kind give the same bits. Frames of the one-workgroup and of the radix depth
sort, near, across 8192 and far, on buffers that grow; selections over levels of which some are
empty; compaction by masks; overlap pruning, also refused."""
import numpy as np
import pytest

from paper_2408_12894_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NAMES = ("means", "log_scales", "quats", "opacity_logits", "sh")


@pytest.fixture
def both(monkeypatch):
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    direct = render.Renderer(0)
    monkeypatch.setenv("FLOD_COUNT_COPY", "1")
    return direct, render.Renderer(0)


def _same_levels(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert x.n == y.n and x.s_min == y.s_min
        for k in NAMES:
            np.testing.assert_array_equal(getattr(x, k).cpu().numpy(), getattr(y, k).cpu().numpy(), err_msg=k)


def test_frames(both):
    from paper_2408_12894_amd import render
    cam = synth.look_at_camera((0.3, -0.2, -3.8), (0, 0, 0), 400, 300)
    for n, scale in ((300, 1.0), (9000, 1.0), (9000, 1e4), (20_000, 1.0), (8192, 1e4), (30_000, 1e4), (9000, 1.0)):
        print(f"[case] counts both ways, frame of {n}, depths x {scale}", flush=True)
        scene = synth.uniform_scene(n, seed=n, s_mu=-4.0, s_sigma=0.5)
        scene.means[::5] = (scene.means[::5] + (0.0, 0.0, 2.0)) * (1.0, 1.0, scale)
        level = render.GaussianLevel.from_scene(scene)
        out = [r.render_level(level, cam, (0.1, 0.2, 0.3)) for r in both]
        views = [r.view() for r in both]
        for x, y in zip(*out):
            np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())
        assert views[0]["stats"] == views[1]["stats"]
        for k in ("values", "ranges", "tiles_touched"):
            np.testing.assert_array_equal(views[0][k], views[1][k])


@pytest.mark.parametrize("sizes,l_start,l_end", [((3000, 700, 0, 2000, 5000), 1, 5), ((0, 0, 900, 0, 0), 2, 4),
                                                 ((500, 0, 0, 0, 1), 1, 5), ((0, 0), 1, 2)])
def test_selections(both, sizes, l_start, l_end):
    from paper_2408_12894_amd import render
    print(f"[case] counts both ways, levels of {sizes}, {l_start} to {l_end}", flush=True)
    levels = [render.GaussianLevel.from_scene(synth.uniform_scene(n, seed=l, s_min=0.1)) if n
              else render._empty_level(0, 0.1, "cuda") for l, n in enumerate(sizes)]
    bands = [0.9, 0.7, 0.5, 0.3, 0.0][5 - len(sizes):]
    kept = [r.select_compact(levels, l_start, l_end, bands, (0.1, 0.0, -0.2)) for r in both]
    _same_levels(*kept)
    if sum(sizes) > 1000:
        assert 0 < sum(lv.n for lv in kept[0]) < sum(sizes)


def test_compaction_and_pruning(both):
    from paper_2408_12894_amd import _lib, render
    for n in (1, 257, 40_000):
        print(f"[case] counts both ways, compaction and pruning of {n}", flush=True)
        level = render.GaussianLevel.from_scene(synth.uniform_scene(n, seed=n, s_min=0.05))
        mask = torch.as_tensor((np.random.default_rng(n).random(n) < 0.4).astype(np.uint8)).cuda()
        _same_levels(*([r.compact(level, mask)] for r in both))
        kept = [r.overlap_prune(level, 0.03, with_d_avg=True) for r in both]
        for x, y in zip(*kept):
            np.testing.assert_array_equal(x.cpu().numpy() if hasattr(x, "cpu") else x, y.cpu().numpy() if hasattr(y, "cpu") else y)
        assert kept[0][1] == int(kept[0][0].sum())
    level.means.mul_(0.01)
    dense = render.GaussianLevel(*(torch.cat([getattr(level, k)] * 8) for k in NAMES), s_min=0.05)
    for r in both:
        with pytest.raises(_lib.FlodError) as e:
            r.overlap_prune(dense, 10.0)
        assert e.value.status == _lib.FLOD_ERR_UNSUPPORTED
