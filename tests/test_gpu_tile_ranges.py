"""The tiles' list ranges by workgroups of 2,048 tiles, and the blend's tile order made beside the
lists: frames of tile counts around whole workgroups against the oracle, and a frame that nothing
shows in, whose order is made by itself."""
import pytest

from paper_2408_12894_amd import synth
from test_gpu_tilebin import _check, _renderer

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [(16, 16), (368, 1424), (1024, 512), (48, 10928), (272, 3856), (1040, 1008)]   # 1, 2047, 2048, 2049, 4097, 4095


@pytest.mark.parametrize("w,h", SIZES)
def test_ranges_around_whole_workgroups(w, h):
    print(f"[case] tile ranges {w}x{h}", flush=True)
    _check(_renderer(), synth.uniform_scene(700, seed=33, s_mu=-3.0, s_sigma=0.6), w, h)


@pytest.mark.parametrize("w,h", SIZES)
def test_order_without_candidates(w, h):
    """Every tile is drawn, also after a frame of another size left its order behind."""
    from paper_2408_12894_amd import render
    print(f"[case] empty frame {w}x{h}", flush=True)
    r = _renderer()
    look = ((0.3, 0.2, -3.6), (0.0, 0.0, 0.0))
    r.render_level(render.GaussianLevel.from_scene(synth.uniform_scene(50, seed=3)), synth.look_at_camera(*look, 320, 240),
                   (0.0, 0.0, 0.0))
    for n_empty in (0, 5):   # none, and some that lie behind the camera
        scene = synth.uniform_scene(n_empty, seed=4) if n_empty else None
        if scene is None:
            level = render._empty_level(0, 0.0, "cuda")
        else:
            scene.means[:] = (0.0, 0.0, -9.0)
            level = render.GaussianLevel.from_scene(scene)
        out = r.render_level(level, synth.look_at_camera(*look, w, h), (0.25, 0.5, 0.75))
        torch.cuda.synchronize()
        image = out[0].cpu()
        for c, v in enumerate((0.25, 0.5, 0.75)):
            assert bool((image[c] == v).all())
        assert bool((out[1] == 1.0).all()) and bool((out[2] == 0).all())
