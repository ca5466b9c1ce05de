"""Which product of the channels' dL/dalpha is rounded.

dL/dalpha = T C + T E (C: the colours' share, E: the extended channels') is one product,
rounded, and a fused multiply-add: fma(T, C, round(T E)).  The footprint sums keep these
bits, since a flat splat seen edge-on amplifies their rounding in its scale gradient.  With
C = -E exactly only the rounding is left, round(T E) - T E, and with the products the
other way round its exact negative, term by term: the sign of the opacity's gradient tells
which it is.  One splat over a 64x64 view, where T = (1 - alpha) rcp(1 - alpha) is 1 or a
few units in the last place off."""
from types import SimpleNamespace

import numpy as np
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("e", [1.2, 1.25, 1.5, 1.75, 1.9])
@pytest.mark.parametrize("pad", [None, 2000, 3000])
def test_the_channels_product_is_rounded(e, pad):
    """pad: a view beside it that brings the tiles to four waves (all, the longest)."""
    import torch
    from paper_2411_09156_amd import Rasterizer, RasterSettings, Splats
    log(f"[gpu] channel rounding E={e} pad={pad}")
    w = 64
    cams = [SimpleNamespace(width=s, height=s if s == w else 500, fx=60.0, fy=60.0, cx=s / 2, cy=w / 2,
                            viewmat=[[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, 1, 4.0]], campos=(0.0, 0.0, -4.0))
            for s in ([w, pad] if pad else [w])]
    sp = Splats(*(torch.tensor(x, dtype=torch.float32, device="cuda") for x in
                  ([[0.013], [0.021], [0.0]], [[0.5], [0.6], [0.4]], [[1.0], [0.0], [0.0], [0.0]], [0.8], [2.0],
                   [[0.0], [0.0], [0.0]])))
    rast = Rasterizer(cams, RasterSettings())
    f = rast.forward(sp, channels=True)
    assert 1000 < int((f["n_contrib"][:w * w] > 0).sum()) < w * w
    e = float(np.float32(e))
    up, up_alpha = torch.zeros(3 * rast.n_pixels, device="cuda"), torch.zeros(rast.n_pixels, device="cuda")
    up[:w * w] = -2.0 * e  # the splat's colour is exactly 0.5 over a black background
    up_alpha[:w * w] = e
    ws = rast.render_bwd_tiles(f["proj"], f["bins"], 1, f["final_T"], f["n_contrib"], up, dL_dalpha=up_alpha,
                               dL_ddepth=torch.zeros_like(up_alpha))
    g = rast.project_bwd(sp, f["proj"], f["bins"], ws, want_grad2d=True)["grad2d"][:12].tolist()
    assert -1e-4 < g[5] < 0.0, g  # opacity: some thousand terms of at most 2^-24
