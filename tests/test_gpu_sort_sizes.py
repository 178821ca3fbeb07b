"""The depth order where the radix sort's workgroups change from 2048 to 3072 keys (4,194,304 candidates) and to
4096 (33,554,432): the tile lists against the oracle's sorted instance list, bit-exact, with depths below 8192
(three passes) and on both sides of it (four)."""
import numpy as np
import pytest

import oracle
from paper_2408_12894_amd import synth
from parity import check_instances, check_keys

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,far,shown", [((4 << 20) - 1, False, 2), (4 << 20, False, 2), ((4 << 20) + 5000, True, 2),
                                         (32 << 20, False, 50)])
def test_order_around_the_larger_workgroups(n, far, shown):
    """shown: one candidate in this many is opaque enough to be rendered."""
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[case] depth sort n={n} far={far}", flush=True)
    rng = np.random.default_rng(17)
    means = rng.uniform(-3.0, 3.0, (n, 3)).astype(np.float32)
    if far:
        p = np.abs(rng.normal(size=(2000, 3))) * (0.0, 0.0, 3e4)
        means[::n // 2000][:2000] = p[: len(means[::n // 2000][:2000])].astype(np.float32)
    logits = np.full(n, -20.0, np.float32)
    logits[rng.integers(0, shown, n) == 0] = 0.0
    logits[::n // 2000] = 0.0
    arrays = [means, np.full((n, 3), -8.0, np.float32), np.tile(np.float32([0.5, 0.5, -0.5, 0.5]), (n, 1)), logits]
    cam = synth.look_at_camera((0.0, 0.0, -3.5), (0.0, 0.0, 0.0), 320, 240)
    r = render.Renderer(0)
    level = render.GaussianLevel(*[torch.from_numpy(a).cuda() for a in arrays], torch.zeros((n, 16, 3), device="cuda"), 0.0)
    r.render_level(level, cam)
    torch.cuda.synchronize()
    view = r.view()
    k = oracle.keys(*arrays, 0.0, cam)
    assert (k["depth_bits"][k["visible"] != 0] >= np.float32(8192.0).view(np.uint32)).any() == far
    check_keys(view, k)
    check_instances(view, k)
