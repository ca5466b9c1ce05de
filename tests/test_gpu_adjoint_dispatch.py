"""The 16x16 adjoint's ways of sharing tiles between 4,096 and 32,768 tiles: all tiles by
four waves up to 5,500, then the longest ones; with the extended channels one wave each
above 12,288 tiles where no view has four times another's pixels.  A view's screen-space
gradients are the same to the bit in batches on each side of these lines."""
import numpy as np
import pytest

import gesr_inputs as gi
from tests.gpu_util import log, splats_of

pytestmark = pytest.mark.gpu

W, H = 1100, 1000  # 4,347 tiles
# views beside the first: none; some that bring the sum over 5,500 and 12,288 tiles with
# resolutions within a factor of four; a small one besides
BATCHES = [[], [(600, 600)], [(1200, 1000)], [(1500, 1100), (900, 800)], [(1500, 1100), (900, 800), (40, 30)]]


@pytest.mark.parametrize("channels", [False, True])
def test_rows_agree_across_the_lines(channels):
    import torch
    from paper_2411_09156_amd import Rasterizer, RasterSettings
    rng = np.random.default_rng([460, 0])
    cams = [gi.look_at((0.1, 0.0, -4.0), width=W, height=H)]
    scene = gi._uniform_cube_scene("lines", rng, 5000, cams)
    sp, n = splats_of(scene), 5000
    gen = torch.Generator(device="cuda").manual_seed(13)
    up = [torch.randn(k * W * H, generator=gen, device="cuda") for k in (3, 1, 1)]
    ref, tiles = None, []
    for extra in BATCHES:
        views = cams + [gi.look_at((0.0, 0.2 * i, -4.0), width=w, height=h) for i, (w, h) in enumerate(extra)]
        log(f"[gpu] adjoint dispatch: {len(views)} views, channels {channels}")
        rast = Rasterizer(views, RasterSettings(sh_degree=scene.sh_degree))
        proj = rast.project(sp)
        bins = rast.bin(proj, n)
        f = rast.render_fwd(proj, bins, n, channels=channels)
        d = [torch.cat([u, torch.full((k * (rast.n_pixels - W * H),), 0.25, device="cuda")]) for u, k in zip(up, (3, 1, 1))]
        ws = rast.render_bwd_tiles(proj, bins, n, f["final_T"], f["n_contrib"], d[0],
                                   dL_ddepth=d[1] if channels else None, dL_dalpha=d[2] if channels else None)
        rows = rast.project_bwd(sp, proj, bins, ws, want_grad2d=True)["grad2d"][:n * 12].cpu().numpy()
        tiles.append(bins["total_tiles"])
        if ref is None:
            ref = rows
            assert np.abs(ref).max() > 0
        np.testing.assert_array_equal(rows, ref, err_msg=str(extra))
    assert tiles[0] <= 5500 < tiles[1] < tiles[2] <= 12288 < tiles[3] < tiles[4] <= 28672
