"""The blend backward's ways of walking a tile (four or two waves per quarter, one wave per tile),
chosen by the frame's tiles: the same scene with the same upstream gradient in the part that all
frames show gives the same gradients.

Tolerance: the sums' order differs. A gradient is a sum of at most some 1e4 FP32 terms per Gaussian,
so it moves by about sqrt(1e4) 2^-24 = 6e-6 of the terms' size; 1e-4 of the array's largest value
leaves room for terms that cancel."""
import dataclasses

import numpy as np
import pytest

from paper_2408_12894_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

W, H = 500, 500


def _grads(scene, cam, dimg):
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = render.Renderer(0)
    level = render.GaussianLevel.from_scene(scene)
    r.render_level(level, cam, (0.1, 0.2, 0.3))
    full = torch.zeros((3, cam.height, cam.width), device="cuda")
    full[:, :H, :W] = dimg
    g = r.backward(level, full)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy().astype(np.float64) for k, v in g.items()}


@pytest.mark.parametrize("n,s_mu,logit", [(1, -2.0, 1.0), (700, -2.5, 2.0), (6000, -3.5, -1.0), (3000, -1.5, -3.0)])
def test_ways_agree(n, s_mu, logit):
    """Frames of 1024 tiles (four waves), 1056 and 2961 (two), 3243 (one per tile): single entries,
    lists of some and of hundreds of entries, opaque and faint."""
    print(f"[case] backward ways n={n} s_mu={s_mu}", flush=True)
    scene = synth.uniform_scene(n, seed=96, s_mu=s_mu, s_sigma=0.5, extent=0.6)
    scene.opacity_logits[:] += np.float32(logit)
    if n == 1:
        scene.means[:] = np.float32(0.1)
    cam = synth.look_at_camera((0.3, -0.2, -3.6), (0.0, 0.0, 0.0), W, H)
    dimg = torch.as_tensor(np.random.default_rng(97).normal(size=(3, H, W)).astype(np.float32)).cuda()
    ref = _grads(scene, cam, dimg)
    assert all(np.abs(v).max() > 0.0 for v in ref.values())
    for w, h in ((520, 500), (1000, 740), (1100, 740)):
        got = _grads(scene, dataclasses.replace(cam, width=w, height=h), dimg)
        for k in ref:
            np.testing.assert_allclose(got[k], ref[k], rtol=0, atol=1e-4 * np.abs(ref[k]).max(), err_msg=f"{k} {w}x{h}")
