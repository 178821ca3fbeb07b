"""The forward blend of frames of few tiles reads each group of eight entries before it takes the one
in front of it. Lists of lengths around whole groups, pairs of groups and staged batches, drawn
in a frame of few tiles and in one of 2,925 (groups taken as they are read): the same pixels, bit
for bit."""
import dataclasses

import numpy as np
import pytest

from paper_2408_12894_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _render(scene, cam):
    from paper_2408_12894_amd import render
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nbl = torch.empty((cam.height, cam.width), dtype=torch.int32, device="cuda")
    r = render.Renderer(0)
    level = render.GaussianLevel.from_scene(scene)
    out = r.render_level(level, cam, (0.1, 0.2, 0.3), n_blended=nbl)
    r.keep_backward_state(False)
    lean = r.render_level(level, cam, (0.1, 0.2, 0.3))
    torch.cuda.synchronize()
    for a, b in zip(out, lean):
        np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
    return [t.cpu().numpy() for t in (*out, nbl)]


@pytest.mark.parametrize("logit", [-4.5, 1.0])   # walked to the end of the list; stopped inside it
@pytest.mark.parametrize("n", [1, 7, 8, 9, 15, 16, 17, 24, 25, 255, 256, 257, 265, 520])
def test_lists_around_whole_groups(n, logit):
    print(f"[case] blend ahead n={n} logit={logit}", flush=True)
    scene = synth.uniform_scene(n, seed=17, s_mu=-0.5, s_sigma=0.1)
    # every Gaussian over the middle of the frame, so that its tiles list all of them
    scene = dataclasses.replace(scene, means=(0.05 * scene.means).astype(np.float32),
                                opacity_logits=np.full_like(scene.opacity_logits, logit))
    small = synth.look_at_camera((0.1, -0.1, -3.6), (0.0, 0.0, 0.0), 112, 80)
    large = dataclasses.replace(small, width=1040, height=720)   # the same pixels in its upper left part
    a, b = _render(scene, small), _render(scene, large)
    assert a[3].max() == n if logit < 0 else a[3].max() > 0
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y[..., :80, :112])
