"""Surface points with other sample counts than 32 (a tail that is switched off, an odd
count, the fewest), against the FP64 oracle as with 32."""
import numpy as np
import pytest

import oracle
from tests import test_gpu_surface as base
from tests.gpu_util import f32, oracle_rec, run_gpu
from tests.test_gpu_parity import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_samples", [2, 8, 9, 31])
def test_other_sample_counts(n_samples):
    import torch
    scene, st = _case("plain-2k")
    g = run_gpu(scene, st)
    rast, sp, out = g["torch"]
    ext = rast.render_fwd(out["proj"], out["bins"], scene.n, channels=True)
    P = scene.n_pixels
    alpha = f32(ext["alpha"])[:P]
    pick = np.random.default_rng(n_samples).choice(np.nonzero(alpha >= 0.3)[0], 1203, replace=False).astype(np.int64)
    kw = dict(n_samples=n_samples, level=base.LEVEL, span=base.SPAN, min_alpha=base.MIN_ALPHA)
    res = rast.surface_points(sp, out["proj"], out["bins"], ext["depth"], ext["alpha"],
                              torch.as_tensor(pick.astype(np.int32)), **kw)
    torch.cuda.synchronize()
    pts, nrm = f32(res["points"]), f32(res["normals"])
    dom = res["dominant"].cpu().numpy().view(np.uint32).astype(np.int64)
    rec = oracle_rec(g["rec"])
    _, vals, ranges = oracle.bin_instances(scene.n, scene.cameras, g["tile_rect"], g["tiles_touched"],
                                           g["depth_key"], st, rec)
    ref = oracle.surface_points(scene, rec, vals, ranges, f32(ext["depth"])[:P].astype(np.float64),
                                alpha.astype(np.float64), pick, st, **kw)
    m = ref["margins"]
    ok = ~((m[:, 2] < 1e-6) | ((ref["dominant"] >= 0) & (m[:, 0] < 1e-3)) | ((ref["valid"] == 1) & (m[:, 1] < 1e-3)))
    assert ok.mean() > 0.9
    gv, rv = pts[:, 3] == 1.0, ref["valid"] == 1
    np.testing.assert_array_equal(gv[ok], rv[ok])
    has = ok & (ref["dominant"] >= 0)
    np.testing.assert_array_equal(dom[has], ref["dominant"][has])
    for r in np.nonzero(ok & gv & rv)[0]:
        h = 2 * base.SPAN * base._sigma(scene, st, ref["dominant"][r], base._ray_dir(scene, pick[r])) / (n_samples - 1)
        assert abs(float(nrm[r, 3]) - ref["t_star"][r]) / h <= 1e-3, r
        cosang = float(np.dot(nrm[r, :3].astype(np.float64), ref["normals"][r]))
        assert float(np.arccos(np.clip(cosang, -1.0, 1.0))) <= 1e-3, r
