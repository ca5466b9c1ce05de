"""Surface points do not depend on which rays share a group of eight: pixels in a shuffled
order (rays of several views and tiles, lists of different lengths, rays that are not
taken) give each pixel's results of the tile-grouped order to the bit."""
import numpy as np
import pytest

import gesr_inputs as gi
from tests.gpu_util import log, splats_of

pytestmark = pytest.mark.gpu

_STATE = {}


def _state():
    import torch
    from paper_2411_09156_amd import Rasterizer, RasterSettings
    if not _STATE:
        scene = gi.make_workload(2, n_override=6000)
        cams = [gi.look_at((0.0, 0.0, -4.0), width=200, height=150), gi.look_at((3.0, 0.5, -2.5), width=64, height=90)]
        rast, sp = Rasterizer(cams, RasterSettings(sh_degree=scene.sh_degree)), splats_of(scene)
        f = rast.forward(sp, channels=True)
        pix = torch.arange(0, rast.n_pixels, 7, device="cuda", dtype=torch.int32)
        _STATE.update(rast=rast, sp=sp, f=f, pix=pix)
    return _STATE


@pytest.mark.parametrize("samples", [2, 7, 8, 9, 16, 17, 24, 31, 32])
@pytest.mark.parametrize("count", [1, 13, None])
def test_order_of_pixels(samples, count):
    import torch
    log(f"[gpu] surface points in two orders, {samples} samples, {count} rays")
    s = _state()
    rast, f, pix = s["rast"], s["f"], s["pix"][:count]
    perm = torch.as_tensor(np.random.default_rng([450, samples]).permutation(pix.numel()), device="cuda")

    def call(p):
        return rast.surface_points(s["sp"], f["proj"], f["bins"], f["depth"], f["alpha"], p, n_samples=samples)

    a, b = call(pix), call(pix[perm])
    if count is None:
        assert 100 < int((a["points"][:, 3] > 0).sum()) < pix.numel()
    for k in a:
        assert torch.equal(a[k][perm], b[k]), k
