"""The 16x16 renderers' ways of sharing a tile among waves give the same bits.

The forward takes a tile with four waves (one 8x8 quadrant each, only the
records that can reach it) or with one; the counting forward always with one.
The adjoint takes a tile with eight waves, four or one.
Tile counts on both sides of the dispatch rules, ragged and one-pixel views,
thin splats (the quadrant's footprint test at its most sheared), beta below 2,
lists that end mid-batch and pixels that terminate."""
import numpy as np
import pytest

import gesr_inputs as gi
import oracle
from tests.gpu_util import splats_of

pytestmark = pytest.mark.gpu


def _needles(n=700):
    rng = np.random.default_rng([400, 0])
    means = rng.uniform(-1.0, 1.0, (n, 3))
    ls = np.stack([rng.uniform(-2.5, -1.0, n), rng.uniform(-10.0, -6.0, n), rng.uniform(-10.0, -6.0, n)], 1)
    return gi._finish("needles", rng, means, ls, gi._random_quats(rng, n), rng.uniform(0.7, 4.0, n),
                      gi._sh_coeffs(rng, n, 0), 0, gi.ring_cameras(2, [(333, 215), (64, 48)]))


def _opaque(n=3000):
    s = gi.tiny_scene(5, n=n, width=90, height=70, deg=0, spread=0.5)
    s.opacities[:] = 0.98
    return s


def _wide(n=4000):
    """More than 8,192 tiles: the leading ones with four waves, the rest with one."""
    rng = np.random.default_rng([401, 0])
    cams = [gi.look_at((0.0, 0.0, -4.0), width=1800, height=1300), gi.look_at((0.5, 0.3, -4.0), width=37, height=19)]
    return gi._uniform_cube_scene("wide", rng, n, cams)


SCENES = {
    "ragged": lambda: gi.ragged_scene(1),
    "one-splat": lambda: gi.tiny_scene(3, n=1, deg=0),
    "plain": lambda: gi.make_workload(1),
    "needles": _needles,
    "opaque": _opaque,
    "wide": _wide,
    "drt-20k": lambda: gi.make_workload(3, n_override=20_000),
}


def _rast(scene, **kw):
    from paper_2411_09156_amd import Rasterizer, RasterSettings
    return Rasterizer(scene.cameras, RasterSettings(sh_degree=scene.sh_degree, bg=(0.2, 0.1, 0.3), **kw))


@pytest.mark.parametrize("name", list(SCENES))
@pytest.mark.parametrize("channels", [False, True])
def test_forward_paths_agree_bitwise(name, channels):
    import torch
    scene = SCENES[name]()
    rast, sp = _rast(scene), splats_of(scene)
    proj = rast.project(sp)
    bins = rast.bin(proj, sp.n)
    outs = []
    for counts in (True, False):
        f = rast.render_fwd(proj, bins, sp.n, counts=counts, channels=channels)
        torch.cuda.synchronize()
        o = {k: f[k].cpu().numpy() for k in ("image", "final_T", "n_contrib") + (("depth", "alpha") if channels else ())}
        o["tile_work"] = bins["tile_work"].cpu().numpy().copy()
        outs.append(o)
    for k in outs[0]:
        np.testing.assert_array_equal(outs[0][k], outs[1][k], err_msg=k)
    if not channels:
        v1 = _rast(scene, variant=1)
        f = v1.render_fwd(proj, v1.bin(proj, sp.n), sp.n)
        for k in ("image", "final_T", "n_contrib"):
            np.testing.assert_array_equal(f[k].cpu().numpy(), outs[0][k], err_msg=k)


@pytest.mark.parametrize("name", [k for k in SCENES if k != "wide"])
@pytest.mark.parametrize("channels", [False, True])
def test_adjoint_paths_agree_bitwise(name, channels):
    """The adjoint takes every tile with eight waves up to 2,048 tiles (rounds of eight
    records up to 512, of four beyond), with four up to
    4,096, the worklist's first 256 with four up to 32,768 and none above: a view's
    screen-space gradients are the same alone and beside a view that brings the batch
    to each."""
    import copy

    import torch
    scene = SCENES[name]()
    n, V = scene.n, scene.n_views
    sp = splats_of(scene)
    gen = torch.Generator(device="cuda").manual_seed(11)
    P = scene.n_pixels
    up = [torch.randn(k, generator=gen, device="cuda") for k in (3 * P, P, P)]
    ref, tiles = None, []
    for pad in (None, (480, 480), (768, 720), (1500, 1100), (4200, 2200)):
        s = copy.copy(scene)
        s.cameras = list(scene.cameras) + ([gi.look_at((0.0, 0.0, -4.0), width=pad[0], height=pad[1])] if pad else [])
        rast = _rast(s)
        proj = rast.project(sp)
        bins = rast.bin(proj, n)
        f = rast.render_fwd(proj, bins, n, channels=channels)
        Q = rast.n_pixels
        dL = [torch.zeros(k, device="cuda") for k in (3 * Q, Q, Q)]
        for d, u in zip(dL, up):
            d[:u.numel()] = u
        if pad:
            dL[0][3 * P:] = 0.25
        ws = rast.render_bwd_tiles(proj, bins, n, f["final_T"], f["n_contrib"], dL[0],
                                   dL_ddepth=dL[1] if channels else None, dL_dalpha=dL[2] if channels else None)
        g = rast.project_bwd(sp, proj, bins, ws, want_grad2d=True)["grad2d"][:n * V * 12].cpu().numpy()
        tiles.append(bins["total_tiles"])
        if ref is None:
            ref = g
            assert np.abs(g).max() > 0
        np.testing.assert_array_equal(g, ref, err_msg=str(pad))
    assert 512 < tiles[1] and 2048 < tiles[2] and 4096 < tiles[3] <= 32768 < tiles[4]
    if tiles[0] <= 1100:
        assert tiles[1] <= 2048 and tiles[2] <= 4096


def _giant():
    s = gi.tiny_scene(8, n=40, width=700, height=520, deg=1)
    s.scales[::2] = np.float32(0.9)  # half of the pairs over hundreds of instance slots
    return s


@pytest.mark.parametrize("name", ["ragged", "one-splat", "needles", "opaque", "drt-20k", "giant"])
def test_gradients_with_and_without_all_rows(name):
    """Pairs that no tile reached have no row of screen-space gradients unless the
    caller asks for them: the parameter gradients are the same either way."""
    import torch
    scene = _giant() if name == "giant" else SCENES[name]()
    rast, sp = _rast(scene), splats_of(scene)
    f = rast.forward(sp)
    dL = torch.randn(3 * rast.n_pixels, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    dL[:dL.numel() // 2] = 0.0  # many tiles without a gradient
    out = []
    for rows in (False, True):
        ws = rast.alloc_workspace(sp.n, f["bins"]["m_cap"])
        ws.fill_(0xFF)  # NaN wherever a row or partial is not written
        rast.render_bwd_tiles(f["proj"], f["bins"], sp.n, f["final_T"], f["n_contrib"], dL, workspace=ws)
        g = rast.project_bwd(sp, f["proj"], f["bins"], ws, want_grad2d=rows)
        out.append({k: v.cpu().numpy() for k, v in g.items()})
    assert np.isfinite(out[1]["grad2d"]).all()
    for k in out[0]:
        assert np.isfinite(out[0][k]).all(), k
        np.testing.assert_array_equal(out[0][k], out[1][k], err_msg=k)


def test_sums_agree_on_both_sides_of_the_pair_count():
    """Above 262,144 pairs a wave of the segmented sum looks 64 of them up, below 16:
    a batch of three views (270,000 pairs) gives each view's rows as the view alone."""
    import copy

    import torch
    rng = np.random.default_rng([402, 0])
    cams = [gi.look_at((0.4 * i, 0.1, -4.0), width=w, height=h) for i, (w, h) in enumerate([(190, 150), (64, 48), (33, 90)])]
    scene = gi._uniform_cube_scene("pairs", rng, 90_000, cams)
    scene.scales[::9] *= 6.0  # pairs over hundreds of instance slots
    sp = splats_of(scene)
    outs = []
    for views in ([0, 1, 2], [0], [1], [2]):
        s = copy.copy(scene)
        s.cameras = [cams[v] for v in views]
        rast = _rast(s)
        f = rast.forward(sp)
        dL = torch.cat([torch.full((3 * cams[v].width * cams[v].height,), 0.1 * (v + 1), device="cuda") for v in views])
        g = rast.render_bwd(sp, f["proj"], f["bins"], f["final_T"], f["n_contrib"], dL, want_grad2d=True)
        outs.append(g["grad2d"][:len(views) * sp.n * 12].cpu().numpy())
    assert np.abs(outs[0]).max() > 0
    np.testing.assert_array_equal(outs[0], np.concatenate(outs[1:]))
