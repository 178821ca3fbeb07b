"""The backward of small frames against 64 bits: sums over many (quarter of a tile, Gaussian) terms.

Sixteen Gaussians that each cover the whole frame, an upstream gradient of one in every channel: a
Gaussian's colour gradient is then the plain sum of its blend weights, all positive, over some 4e3
(512x512) or 9e3 (768x768) terms of a wave's 64 pixels. What a term's own FP32 arithmetic leaves in
it: the roundings that differ between pixels average out over 2.6e5 of them; those of a Gaussian's own
staged values are the same in all: its opacity (2 ulp of the exponential), log2 of it (at most 4 in
size) and the conic (a q of at most 4 here), each within 2^-24 of its size and carried to alpha by
ln 2 or 1/2, 4e-7 together, and half of that again for the transmittance of those in front (their
weights are small). Adding the terms up in FP32 instead leaves about
2^-24 sqrt(n / 3): 2e-6 and 3e-6 here. The bound is 1e-6 of the sum."""
import numpy as np
import pytest

import oracle
from paper_2408_12894_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _scene():
    scene = synth.uniform_scene(16, seed=41, extent=0.15)
    rng = np.random.default_rng(42)
    scene.log_scales[:] = rng.uniform(0.5, 1.0, scene.log_scales.shape).astype(np.float32)
    scene.opacity_logits[:] = rng.uniform(-3.0, -1.5, scene.opacity_logits.shape).astype(np.float32)
    scene.sh[:] = (0.1 * rng.random(scene.sh.shape)).astype(np.float32)
    scene.sh[:, 0] = 1.0   # no colour is clamped
    return scene


@pytest.mark.parametrize("size", [512, 768])
def test_colour_sums(size):
    """1,024 tiles (four waves per quarter tile) and 2,304 (two)."""
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[case] backward colour sums {size}x{size}", flush=True)
    scene = _scene()
    cam = synth.look_at_camera((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), size, size)
    bg = np.zeros(3, np.float32)
    r = render.Renderer(0)
    level = render.GaussianLevel.from_scene(scene)
    r.render_level(level, cam, bg, 0)
    got = r.backward(level, torch.ones((3, size, size), device="cuda"))["sh"][:, 0].cpu().numpy().astype(np.float64)
    order = oracle.depth_order(oracle.keys(*scene.arrays()[:4], scene.s_min, cam))
    pix = oracle.all_pixels(size, size)
    ref = oracle.grad(order, *scene.arrays()[:4], scene.s_min, scene.sh, 0, cam, bg, pix, np.ones((pix.shape[0], 3)))
    ref = ref["sh"][:, 0]
    assert ref.min() > 0.0
    err = np.abs(got - ref) / ref
    print(f"[sums] {size}: largest relative error {err.max():.2e}, RMS {np.sqrt((err * err).mean()):.2e}", flush=True)
    assert err.max() <= 1e-6
