"""The blend's per-quadrant entry lists against the oracle: a pixel blends what the oracle blends, up
to the last Gaussian and the count, where dropping an entry for a quadrant could go wrong:
Gaussians of a pixel or less on the quadrants' borders, long thin ones across their corners, and
opacities near the alpha floor, whose support ends inside the footprint. Tolerances in parity.py."""
import numpy as np
import pytest

from paper_2408_12894_amd import synth
from test_gpu_forward import full_parity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _scene(kind, n, seed):
    rng = np.random.default_rng(seed)
    sc = synth.uniform_scene(n, seed=seed, s_mu=-5.0, s_sigma=0.4, extent=1.0)
    if kind == "specks":
        sc.log_scales[:] = np.float32(-7.0)
        sc.opacity_logits[:] = np.float32(3.0)
    elif kind == "needles":
        sc.log_scales[:] = np.float32(-7.0)
        sc.log_scales[:, 0] = rng.uniform(-4.0, -1.5, n).astype(np.float32)
        sc.opacity_logits[:] = rng.uniform(-2.0, 1.0, n).astype(np.float32)
    else:   # faint: opacities from the floor to three times it
        sc.log_scales[:] = rng.uniform(-5.0, -1.0, (n, 3)).astype(np.float32)
        o = rng.uniform(1.001, 3.0, n) / 255.0
        sc.opacity_logits[:] = np.log(o / (1.0 - o)).astype(np.float32)
    return sc


@pytest.mark.parametrize("kind", ["specks", "needles", "faint"])
@pytest.mark.parametrize("w,h,s_min,sample", [(160, 144, 0.0, None), (1100, 1000, 0.0, (6000, 3000, 5)),
                                              (1100, 1000, 0.02, (6000, 3000, 6))])
def test_quadrants_blend_what_the_oracle_blends(kind, w, h, s_min, sample):
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[case] quadrants {kind} {w}x{h} s_min={s_min}", flush=True)
    scene = _scene(kind, 1500, 95)
    scene.s_min = s_min
    cam = synth.look_at_camera((0.3, -0.2, -2.9), (0.0, 0.0, 0.0), w, h)
    full_parity(render.Renderer(0), scene, cam, (0.1, 0.2, 0.3), sample=sample, label=kind)
