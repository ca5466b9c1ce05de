"""The binning's ways of sorting and scanning give the same lists.

The (view, depth) sort takes a view in LDS (up to 4,096 splats, 1, 2 or 4 per
thread), by blocks of 1,024, 2,048 or 4,096 keys that find their offsets
themselves, or with a scan between the kernels of a pass; the tile lists of up
to 16,384 tiles come from one workgroup (1, 4 or 16 tiles per thread).  Both
sides of every rule, with equal depths and splats behind the camera, against
the order of the keys and the narrower digits' general sort."""
import numpy as np
import pytest

import gesr_inputs as gi
from tests.gpu_util import splats_of, u32

pytestmark = pytest.mark.gpu


def _scene(n, sizes):
    rng = np.random.default_rng([410, n])
    cams = [gi.look_at((0.3 * i, 0.2, -4.0), width=w, height=h) for i, (w, h) in enumerate(sizes)]
    s = gi._uniform_cube_scene("bins", rng, n, cams)
    s.means[n // 2:] = s.means[:n - n // 2]  # equal depths
    s.means[5::7, 2] -= 40.0                 # behind the cameras
    return s


def _bins(scene, bits):
    import torch
    from paper_2411_09156_amd import Rasterizer, RasterSettings
    rast, sp = Rasterizer(scene.cameras, RasterSettings(sh_degree=scene.sh_degree, radix_bits=bits)), splats_of(scene)
    proj = rast.project(sp)
    b = rast.bin(proj, sp.n)
    torch.cuda.synchronize()
    cnt = u32(b["counters"])[:4].copy()
    T, M, vn = b["total_tiles"], int(cnt[3]), scene.n * scene.n_views
    return dict(counters=cnt, val=u32(b["val_sorted"])[:M].copy(), tile=u32(b["tile_sorted"])[:M].copy(),
                ranges=u32(b["ranges"])[:2 * T].reshape(T, 2).copy(), worklist=u32(b["worklist"])[:T].copy(),
                inst_base=u32(b["inst_base"])[:vn].copy(), touched=u32(proj["tiles_touched"])[:vn].copy(),
                depth=u32(proj["depth_key"])[:vn].copy())


@pytest.mark.parametrize("n,sizes", [
    (1, [(16, 16)]), (1024, [(70, 40), (16, 16)]), (1025, [(512, 512)]), (2049, [(512, 513)]),
    (4096, [(300, 200), (90, 33), (1, 1)]), (4097, [(1024, 1024), (16, 16)]), (65_536, [(1024, 1025)]),
    (65_537, [(200, 100), (333, 215)]), (131_073, [(2048, 2048)]), (262_145, [(2048, 2049), (50, 60)]),
], ids=lambda x: str(x) if isinstance(x, int) else f"{len(x)}v")
def test_lists_in_key_order_on_every_path(n, sizes):
    scene = _scene(n, sizes)
    g, narrow = _bins(scene, 8), _bins(scene, 4)
    for k in g:
        np.testing.assert_array_equal(g[k], narrow[k], err_msg=k)
    # the key order: tile, then depth bits, then pair
    val = g["val"].astype(np.int64)
    np.testing.assert_array_equal(np.lexsort((val, g["depth"][val], g["tile"])), np.arange(val.size))
    assert (np.bincount(val, minlength=g["touched"].size) <= g["touched"]).all()  # rectangles, not footprints
    ends = np.cumsum(g["touched"], dtype=np.uint64)
    np.testing.assert_array_equal(g["inst_base"], ends - g["touched"])
    assert g["counters"].tolist() == [int(ends[-1]), 0, int(ends[-1]), val.size]
    T = g["ranges"].shape[0]
    lens = np.bincount(g["tile"], minlength=T)
    first = np.cumsum(lens) - lens
    np.testing.assert_array_equal(g["ranges"], np.where(lens[:, None] > 0, np.stack([first, first + lens], 1), 0))
    np.testing.assert_array_equal(g["worklist"], np.lexsort((np.arange(T), -np.minimum(lens, 0xFFFF))))
