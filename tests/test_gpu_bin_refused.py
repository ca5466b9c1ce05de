"""gesr_bin with GESR_BIN_SYNC whose instances exceed the capacity: the call says how
many there are, the stream is drained when it returns, and the lists, ranges and worklist
of the caller are as they were."""
import ctypes

import pytest

import gesr_inputs as gi
from tests.gpu_util import log, splats_of

pytestmark = pytest.mark.gpu

# one view in LDS and with scans; several views; more than 16,384 tiles
SIZES = [(900, [(200, 150)]), (9000, [(333, 215), (64, 48), (90, 70)]), (5000, [(2100, 2200)])]


def _case(n, sizes, **kw):
    import numpy as np
    from paper_2411_09156_amd import Rasterizer, RasterSettings
    rng = np.random.default_rng([430, n])
    cams = [gi.look_at((0.3 * i, 0.1, -4.0), width=w, height=h) for i, (w, h) in enumerate(sizes)]
    scene = gi._uniform_cube_scene("refused", rng, n, cams)
    rast = Rasterizer(cams, RasterSettings(sh_degree=scene.sh_degree, **kw))
    return rast, splats_of(scene)


def _call(rast, proj, b, n, static=False):
    from paper_2411_09156_amd import _lib
    from paper_2411_09156_amd.rasterizer import _stream
    m = ctypes.c_uint64(0)
    fn = rast.lib.gesr_bin_static if static else rast.lib.gesr_bin
    st = fn(rast.ctx, ctypes.byref(rast._proj_c(proj)), rast.cams_c, rast.V, n, ctypes.byref(rast.st_c),
            ctypes.byref(rast._bins_c(b)), _lib.GESR_BIN_SYNC, ctypes.byref(m), _stream())
    return st, m.value


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("radix_bits", [8, 6])
@pytest.mark.parametrize("n,sizes", SIZES)
def test_refused_call_leaves_the_lists(n, sizes, radix_bits, static):
    import torch
    from paper_2411_09156_amd import _lib
    log(f"[gpu] refused binning n={n} views={len(sizes)} radix={radix_bits} static={static}")
    rast, sp = _case(n, sizes, radix_bits=radix_bits)
    proj = rast.project(sp)
    full = rast.bin(proj, n)
    m = full["M"]
    for m_cap in (m - 1, m // 3):
        b = rast.alloc_bins(n, m_cap)
        b["scratch"].fill_(0xA7)  # counts of an earlier call, say
        kept = {}
        for k in ("tile_sorted", "val_sorted", "ranges", "worklist"):
            b[k].fill_(0x5A5A5A5A)
            kept[k] = b[k].clone()
        torch.cuda.synchronize()
        st, got = _call(rast, proj, b, n, static)
        drained = torch.cuda.current_stream().query()
        assert (st, got) == (_lib.GESR_ERR_CAPACITY, m)
        assert drained
        assert b["counters"][:3].tolist() == [m, 1, m_cap]
        torch.cuda.synchronize()
        for k, v in kept.items():
            assert torch.equal(b[k], v), k
        # the call repeated with room gives the lists of before
        c = rast.alloc_bins(n, m)
        st, got = _call(rast, proj, c, n, static)
        assert (st, got) == (_lib.GESR_OK, m)
        listed = int(full["counters"][3])
        assert torch.equal(c["val_sorted"][:listed], full["val_sorted"][:listed])
        assert torch.equal(c["ranges"], full["ranges"]) and torch.equal(c["worklist"], full["worklist"])
