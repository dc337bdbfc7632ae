"""Backward stage 1 at the sizes its grouping turns on: 16 entries per group, 64
per staging, 256 list positions in a tile's sum table; quads cut by the canvas,
pixels that stop inside a group; the packed accumulation of
bz_render_bwd_scratch against the planes of bz_render_bwd; a NaN in the image
gradient stays with the tiles it reaches."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_2503_16424_amd import bz, scenes
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

GRAD_TOL = 1e-3        # per group, as for every gradient comparison with the oracle
ORDER_TOL = 1e-5       # float atomics in another order


def _strokes(W, H, n, K, opacity, seed=3):
    rng = np.random.default_rng(seed)
    ctrl = rng.uniform(-0.1, 1.1, (n, 4, 2)) * [W, H]
    return scenes.open_curves(W, H, ctrl, rng.uniform(1.5, 4.0, n), rng.uniform(0, 1, (n, 3)),
                              opacity * rng.uniform(0.5, 1.0, n), K)


def _planes_backward(r, dimg):
    """bz_render_bwd (no scratch) on the rasterizer's buffers."""
    bz._check("bz_render_bwd", r.lib.bz_render_bwd(
        C.byref(r.curves), C.byref(r.gauss), C.byref(r.bins), C.byref(r.opts), bz._ptr(dimg),
        r._state_arg(), C.byref(r.grads), bz._stream()))


GROUPS = ("d_ctrl", "d_width", "d_color", "d_opacity")


@pytest.mark.parametrize("state", ["stored", "recompute"])
@pytest.mark.parametrize("W,H", [(8, 8), (21, 13)])
@pytest.mark.parametrize("n,K,opacity", [
    (1, 2, 0.9), (1, 15, 0.02), (1, 16, 0.02), (1, 17, 0.02), (1, 63, 0.02), (1, 64, 0.02),
    (1, 65, 0.02), (1, 129, 0.02), (1, 255, 0.01), (1, 257, 0.01), (3, 101, 0.01),
    (6, 33, 0.6), (9, 40, 1.0)])
def test_group_edges_match_oracle(state, W, H, n, K, opacity):
    import torch
    sc = _strokes(W, H, n, K, opacity)
    img = oracle.forward_backward(sc)["image"]
    tgt = scenes.target_noise(7, W, H).astype(np.float64)
    d = (2.0 * (img - tgt) / img.size).astype(np.float32)
    o = oracle.forward_backward(sc, d.astype(np.float64))
    r = bz.Rasterizer(sc, blend_state=state)
    r.render()
    dimg = torch.as_tensor(d, device="cuda")
    r.backward(dimg)
    got = {k: getattr(r, k).cpu().numpy() for k in GROUPS}
    planes = r.d_gauss_host()
    _planes_backward(r, dimg)
    for k in GROUPS:
        assert rel_l2(got[k], o[k]) <= GRAD_TOL, (k, "scratch")
        assert rel_l2(getattr(r, k).cpu().numpy(), o[k]) <= GRAD_TOL, (k, "planes")
    for v, (a, b) in enumerate(zip(planes.T, r.d_gauss_host().T)):
        assert rel_l2(a, b) <= ORDER_TOL, ("plane", v)


@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 32), (64, 16)])
def test_packed_and_plane_gradients_agree(tile):
    """Many curves and tiles, closed and open, every per-Gaussian plane."""
    import torch
    sc = scenes.mixed(3, 200, 168, 40, 30, K=24, R=20, S_open=3, extent=(4.0, 120.0))
    r = bz.Rasterizer(sc, bz.RenderOptions(tile_w=tile[0], tile_h=tile[1]))
    r.render()
    dimg = torch.as_tensor(scenes.target_noise(5, 200, 168) - 0.5, device="cuda")
    r.backward(dimg)
    a = r.d_gauss_host()
    curves = {k: getattr(r, k).cpu().numpy() for k in GROUPS}
    _planes_backward(r, dimg)
    for v, (x, y) in enumerate(zip(a.T, r.d_gauss_host().T)):
        assert rel_l2(x, y) <= ORDER_TOL, ("plane", v)
    for k in GROUPS:
        assert rel_l2(curves[k], getattr(r, k).cpu().numpy()) <= ORDER_TOL, k


def test_nan_gradient_stays_in_its_tile():
    """A NaN at one pixel of one channel: Gaussians whose support does not
    reach the pixel's tile keep finite gradients."""
    import torch
    sc = scenes.uniform_open(9, 64, 64, 40, 16)
    sc.stroke_w[:] = 1.0
    r = bz.Rasterizer(sc)
    r.render()
    d = scenes.target_noise(5, 64, 64) - 0.5
    d[1, 5, 6] = np.nan
    r.backward(torch.as_tensor(d, device="cuda"))
    g = r.d_gauss_host()
    ranges, ids = r.tile_lists()
    near = np.zeros(sc.n_gauss, bool)
    near[ids[ranges[0, 0]: ranges[0, 1]]] = True
    assert np.isnan(g[near]).any()
    assert np.isfinite(g[~near]).all()


def test_width_gradients_of_long_strokes():
    """Diagonal strokes much longer than wide: the moments along them are hundreds of
    times those across, of which the width's gradient is made.  The step's gradients
    against the stage-by-stage form with its planes in x and y: control points 1e-4, and
    the widths no further off FP64 than that form's (1e-4 at most)."""
    import torch

    import oracle
    from paper_2503_16424_amd import bz, scenes
    from tests.helpers import rel_l2
    sc = scenes.uniform_open(31, 256, 256, 24, 12)
    r = bz.Rasterizer(sc)
    r.render()
    o0 = oracle.forward_backward(sc)
    tgt = scenes.target_noise(3, sc.width, sc.height).astype(np.float64)
    d = 2.0 * (o0["image"] - tgt) / o0["image"].size
    o = oracle.forward_backward(sc, d)
    dt = torch.as_tensor(d.astype(np.float32), device="cuda")
    r.backward(dt)
    got = {k: getattr(r, k).clone() for k in ("d_ctrl", "d_width")}
    planes = r.d_gauss.clone()
    r.backward_gauss(dt)
    assert rel_l2(planes.cpu().numpy(), r.d_gauss.double().cpu().numpy()) <= 1e-5
    r.backward_curves()
    for k in got:
        assert rel_l2(got[k].cpu().numpy(), o[k]) <= max(
            1e-4, 1.5 * rel_l2(getattr(r, k).cpu().numpy(), o[k])), k
    assert rel_l2(got["d_width"].cpu().numpy(), o["d_width"]) <= 1e-4
