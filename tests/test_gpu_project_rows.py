"""Projection of a batch against its views one at a time, to the bit, at splat counts
where the batch's views are shared by rows of workgroups: a row a view, several views a
row, rows without a view, one row."""
import numpy as np
import pytest

import gesr_inputs as gi
from tests.gpu_util import log, splats_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,views,deg", [(1, 32, 0), (255, 5, 1), (257, 32, 2), (20_000, 32, 3), (30_000, 11, 0),
                                         (70_000, 7, 3), (330_000, 3, 1)])
def test_batch_equals_views(n, views, deg):
    import torch
    from paper_2411_09156_amd import Rasterizer, RasterSettings
    log(f"[gpu] projection n={n} views={views} degree={deg}")
    rng = np.random.default_rng([470, n])
    cams = gi.ring_cameras(views, [(40 + 7 * v, 30 + 3 * v) for v in range(views)])
    scene = gi._uniform_cube_scene("rows", rng, n, cams, deg=deg)
    sp = splats_of(scene)
    both = Rasterizer(cams, RasterSettings(sh_degree=deg)).project(sp)
    assert int((both["tiles_touched"] > 0).sum()) > 0 or n == 1
    for v in range(views):
        one = Rasterizer([cams[v]], RasterSettings(sh_degree=deg)).project(sp)
        for k, w in (("rec", 16), ("tiles_touched", 1), ("rect", 2), ("depth_key", 1)):
            a, b = both[k][v * w * n:(v + 1) * w * n], one[k][:w * n]
            assert torch.equal(a.view(torch.int32), b.view(torch.int32)), (k, v)
