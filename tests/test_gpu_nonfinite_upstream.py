"""Upstream gradients that are not finite stay with the splats of their pixels.

A ratio of the extended channels (depth / alpha) has no finite gradient where nothing is
composited, and a loss may overflow at one pixel.  A splat that such a pixel did not
composite keeps its gradient to the bit, however the tile is shared among waves."""
import copy

import numpy as np
import pytest

import gesr_inputs as gi
from tests.gpu_util import log, splats_of
from tests.test_gpu_render_paths import _needles, _rast

pytestmark = pytest.mark.gpu


def _sparse():
    """Few small splats: most pixels of a tile composite none of its list."""
    return gi.tiny_scene(21, n=150, width=200, height=140, deg=0, spread=0.9)


def _rows(rast, sp, f, up, channels):
    ws = rast.render_bwd_tiles(f["proj"], f["bins"], sp.n, f["final_T"], f["n_contrib"], up[0],
                               dL_ddepth=up[1] if channels else None, dL_dalpha=up[2] if channels else None)
    g = rast.project_bwd(sp, f["proj"], f["bins"], ws, want_grad2d=True)
    return g["grad2d"][:rast.V * sp.n * 12].cpu().numpy().reshape(-1, 12)


# a view that brings the batch to each way of sharing the adjoint's tiles (eight waves
# with long and short rounds, four, some, none), and the other tile shapes
FORMS = [(pad, {}, channels) for pad in (None, (480, 480), (768, 720), (1500, 1100), (4200, 2200))
         for channels in (False, True)]
FORMS += [(None, dict(variant=1), False)] + [(None, dict(tile_w=w, tile_h=h), False) for w, h in ((8, 8), (32, 16), (32, 32))]


@pytest.mark.parametrize("scene", [_sparse, _needles])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("pad,settings,channels", FORMS)
def test_empty_pixels_reach_no_splat(scene, value, pad, settings, channels):
    """Non-finite values at every pixel that composited nothing leave all rows as they
    are with zeros there."""
    import torch
    s = scene()
    if pad:
        s = copy.copy(s)
        s.cameras = list(s.cameras) + [gi.look_at((0.0, 0.0, -4.0), width=pad[0], height=pad[1])]
    rast, sp = _rast(s, **settings), splats_of(s)
    log(f"[gpu] non-finite upstream {scene.__name__} {value} {pad} {settings} {channels}")
    f = rast.forward(sp, channels=channels)
    P = rast.n_pixels
    gen = torch.Generator(device="cuda").manual_seed(12)
    up = [torch.randn(k, generator=gen, device="cuda") for k in (3 * P, P, P)]
    empty = f["n_contrib"][:P] == 0
    assert 0 < int(empty.sum()) < P
    image, at = [], 0
    for w, h in rast.views:
        image.append(empty[at:at + w * h].repeat(3))
        at += w * h
    empty = [torch.cat(image), empty, empty]
    zero, bad = ([torch.where(e, torch.full_like(u, x), u) for u, e in zip(up, empty)] for x in (0.0, value))
    want = _rows(rast, sp, f, zero, channels)
    assert np.isfinite(want).all() and np.abs(want).max() > 0
    np.testing.assert_array_equal(_rows(rast, sp, f, bad, channels), want)
