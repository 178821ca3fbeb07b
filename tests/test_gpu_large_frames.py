"""Frames of more than 512 supertiles (above 3840x2160), whose pairs are placed window by window and
counted per column of up to 32 x 256 Gaussians: the tile lists against the oracle, bit-exact, every
tile drawn, and the workspace."""
import numpy as np
import pytest

from paper_2408_12894_amd import synth
from test_gpu_tilebin import SCENES, _check, _renderer

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FINE = dict(seed=85, s_mu=-6.5, s_sigma=1.0, extent=1.5)


@pytest.mark.parametrize("kind,n,w,h", [
    ("fine", 65_536, 4224, 2176), ("fine", 65_537, 4224, 2176),      # 561 supertiles: columns of 256 and of 512
    ("fine", 140_000, 7680, 4320),                                   # 2,040: four windows, columns of 768
    ("fine", 70_000, 16384, 16384),                                  # 16,384: 32 windows
    ("needles", 300, 640, 16384), ("blobs", 30, 650, 16384),         # five and six supertiles a row
    ("blobs", 9, 16384, 640), ("mixed", 257, 9000, 3000),
])
def test_lists_of_large_frames(kind, n, w, h):
    print(f"[case] large frame {kind} n={n} {w}x{h}", flush=True)
    _check(_renderer(), synth.uniform_scene(n, **FINE) if kind == "fine" else SCENES[kind](n), w, h)


@pytest.mark.parametrize("w,h", [(4096, 2048), (4112, 2048), (6000, 6001)])   # 32,768 tiles, 32,896 and 141,000
def test_every_tile_is_drawn(w, h):
    """The tile order by one workgroup and by several."""
    from paper_2408_12894_amd import render
    print(f"[case] tile order {w}x{h}", flush=True)
    r = _renderer()
    cam = synth.look_at_camera((0.4, -0.2, -3.7), (0, 0, 0), w, h)
    level = render.GaussianLevel.from_scene(synth.uniform_scene(2000, seed=86))
    out = (torch.full((3, h, w), float("nan"), device="cuda"), torch.full((h, w), float("nan"), device="cuda"),
           torch.full((h, w), -1, dtype=torch.int32, device="cuda"))
    for _ in range(2):
        r.render_level(level, cam, (0.25, 0.5, 0.75), out=out)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out[0]).all()) and bool((out[1] <= 1.0).all()) and bool((out[2] >= 0).all())


def test_workspace_of_a_large_frame():
    """What a render without backward state holds at 16384x16384, each with the allocator's 25%: some 100
    bytes per candidate, 20 per tile, 290 per supertile, a 4-byte pair count per supertile and column (at
    most 256 columns and their rounding here), 16 bytes per instance or pair. With a count per
    supertile and 256 Gaussians it was twice the bound."""
    from paper_2408_12894_amd import render
    n, side = 200_000, 16384
    print("[case] workspace at 16384x16384", flush=True)
    r = _renderer()
    r.keep_backward_state(False)
    level = render.GaussianLevel.from_scene(synth.uniform_scene(n, **dict(FINE, s_mu=-9.0, s_sigma=0.1)))
    cam = synth.look_at_camera((0.4, -0.2, -3.7), (0, 0, 0), side, side)
    out = (torch.empty((3, side, side), device="cuda"), torch.empty((side, side), device="cuda"),
           torch.empty((side, side), dtype=torch.int32, device="cuda"))
    r.render_level(level, cam, out=out)
    tiles, supers, k = (side // 16) ** 2, (side // 128) ** 2, r.stats()["n_instances"]
    bound = 1.25 * (104 * n + 20 * tiles + (290 + 4 * 264) * supers + 16 * k)
    print(f"  {r.workspace_bytes() / 2**20:.1f} MiB, bound {bound / 2**20:.1f}, K {k}", flush=True)
    assert np.isfinite(bound) and r.workspace_bytes() <= bound
