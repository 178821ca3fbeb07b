"""The L1 + SSIM loss of small and of narrow images, whose workgroups take one step each however few 16 x 16
tiles they have: loss and gradient against the FP64 oracle, with the bounds of the other sizes
(the loss within 1e-12, the gradient within 1e-5 of its largest value and 1e-6 of its own), forward by both
entry points. Three channels of 1,364 rows make 1,023 workgroups of one step, of 1,366 one more than 1,024."""
import ctypes as C

import numpy as np
import pytest

from oracle import ssim as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 4, 4), (1, 16, 16), (3, 17, 16), (64, 5, 3), (3, 500, 16), (1, 4100, 20),
                                   (3, 1364, 1), (3, 1366, 4)])
def test_small_images(shape):
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[case] loss of {shape}", flush=True)
    rng = np.random.default_rng(sum(shape))
    x = rng.random(shape).astype(np.float32)
    y = np.clip(x + 0.2 * rng.normal(size=shape), 0, 1).astype(np.float32)
    r = render.Renderer(0)
    xt = torch.as_tensor(x).cuda().requires_grad_(True)
    yt = torch.as_tensor(y).cuda()
    loss = render.l1_ssim_loss(xt, yt, renderer=r)
    loss.backward()
    lam = float(np.float32(0.2))
    grad = S.loss_grad(x, y, lam)
    assert abs(loss.item() - S.loss(x, y, lam)) <= 1e-12
    assert (np.abs(xt.grad.cpu().numpy() - grad) <= 1e-5 * np.abs(grad).max() + 1e-6 * np.abs(grad)).all()
    lean = torch.empty((), dtype=torch.float64, device="cuda")
    st = r.L.flod_l1_ssim_forward_noalloc(r.ctx, C.c_void_p(xt.data_ptr()), C.c_void_p(yt.data_ptr()), *shape, 0.2,
                                          C.c_void_p(lean.data_ptr()), None, None)
    torch.cuda.synchronize()
    assert st == 0 and lean.item() == loss.item()
