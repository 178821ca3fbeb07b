"""The forward blend's ways of taking a group of entries (branches; 8 or 16 predicated entries),
chosen by the frame's tiles and the levels' scale floors. The same scene drawn as one frame and as
part of a larger one blends the same pixels bit for bit; a colour that is not finite reaches
only the pixels that blend its Gaussian."""
import dataclasses

import numpy as np
import pytest

from paper_2408_12894_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _render(scene, cam, s_min):
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    scene = dataclasses.replace(scene, s_min=s_min)
    nbl = torch.empty((cam.height, cam.width), dtype=torch.int32, device="cuda")
    r = render.Renderer(0)
    out = r.render_level(render.GaussianLevel.from_scene(scene), cam, (0.1, 0.2, 0.3), n_blended=nbl)
    r.keep_backward_state(False)
    lean = r.render_level(render.GaussianLevel.from_scene(scene), cam, (0.1, 0.2, 0.3))
    torch.cuda.synchronize()
    for a, b in zip(out, lean):
        np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
    return [t.cpu().numpy() for t in (*out, nbl)]


@pytest.mark.parametrize("s_min", [0.0, 0.02])
@pytest.mark.parametrize("n", [40, 3000])
def test_small_frame_inside_a_large_one(s_min, n):
    """A frame of 520 x 200 pixels (429 tiles) and one of 1560 x 1080 (6,664) whose upper left part
    shows the same pixels: same focal length and principal point, tiles aligned."""
    print(f"[case] blend ways n={n} s_min={s_min}", flush=True)
    scene = synth.uniform_scene(n, seed=91, s_mu=-3.5, s_sigma=0.8, a_sigma=2.0)
    small = synth.look_at_camera((0.3, -0.2, -3.6), (0.0, 0.0, 0.0), 520, 200)
    # the clamp of the projection's Jacobian follows the frame's half width: keep every mean inside it
    large = dataclasses.replace(small, width=1560, height=1080)
    a, b = _render(scene, small, s_min), _render(scene, large, s_min)
    lim = 1.3 * 0.5 * np.array([520, 200]) / small.fx
    t = scene.means.astype(np.float64) @ small.R.T.astype(np.float64) + small.t
    if not (np.abs(t[:, :2]) < lim * t[:, 2:]).all():
        keep = (np.abs(t[:, :2]) < lim * t[:, 2:]).all(1)
        scene = synth.Scene(*(x[keep] for x in scene.arrays()))
        a, b = _render(scene, small, s_min), _render(scene, large, s_min)
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y[..., :200, :520])


@pytest.mark.parametrize("w,h,s_min", [(128, 96, 0.0), (1600, 1100, 0.05), (1600, 1100, 0.0)])
def test_infinite_colour(w, h, s_min):
    print(f"[case] infinite colour {w}x{h} s_min={s_min}", flush=True)
    scene = synth.uniform_scene(600, seed=92, s_mu=-3.0, s_sigma=0.5)
    cam = synth.look_at_camera((0.1, 0.3, -3.6), (0.0, 0.0, 0.0), w, h)
    ref = _render(scene, cam, s_min)
    bad = scene.copy()
    bad.sh[::97, 0, :] = np.inf
    got = _render(bad, cam, s_min)
    for x, y in zip(got[1:], ref[1:]):
        np.testing.assert_array_equal(x, y)
    finite = np.isfinite(got[0])
    assert 0 < finite.sum() < finite.size
    np.testing.assert_array_equal(got[0][finite], ref[0][finite])
