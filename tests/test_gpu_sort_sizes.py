"""The depth order where the radix sort's workgroups change from 2048 to 4096 keys (2,097,152 candidates):
the tile lists against the oracle's sorted instance list, bit-exact, with depths below 8192 (three
passes) and on both sides of it (four)."""
import numpy as np
import pytest

import oracle
from paper_2408_12894_amd import synth
from parity import check_instances, check_keys

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,far", [((2 << 20) - 1, False), (2 << 20, False), ((2 << 20) + 5000, True)])
def test_order_around_the_large_workgroups(n, far):
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[case] depth sort n={n} far={far}", flush=True)
    rng = np.random.default_rng(17)
    one = synth.uniform_scene(1, seed=17)
    means = rng.uniform(-3.0, 3.0, (n, 3)).astype(np.float32)
    if far:
        p = np.abs(rng.normal(size=(2000, 3))) * (0.0, 0.0, 3e4)
        means[::n // 2000][:2000] = p[: len(means[::n // 2000][:2000])].astype(np.float32)
    scene = synth.Scene(means, np.full((n, 3), -8.0, np.float32), np.broadcast_to(one.quats, (n, 4)).copy(),
                        np.zeros(n, np.float32), np.zeros((n, 16, 3), np.float32), s_min=0.0, meta={})
    cam = synth.look_at_camera((0.0, 0.0, -3.5), (0.0, 0.0, 0.0), 320, 240)
    r = render.Renderer(0)
    r.render_level(render.GaussianLevel.from_scene(scene), cam)
    torch.cuda.synchronize()
    view = r.view()
    k = oracle.keys(*scene.arrays()[:4], scene.s_min, cam)
    assert (k["depth_bits"][k["visible"] != 0] >= np.float32(8192.0).view(np.uint32)).any() == far
    check_keys(view, k)
    check_instances(view, k)
