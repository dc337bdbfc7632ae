"""The optimisation step's one-launch update and copy against torch's (GPU).

One Adam step in FP32 takes about ten roundings, in another order than torch's
passes: moments within 1e-6 relative of |m| + |g| (v: of v), parameters within 2e-6
of the step's size plus two roundings of the parameter.  The copy into the curve
set takes torch's two operations: equal bits.
"""
import ctypes as C

import numpy as np
import pytest

from paper_2503_16424_amd import scenes


def _fitter(optimizer="adam", **kw):
    from paper_2503_16424_amd import bz, optim
    sc = scenes.mixed(3, 120, 72, 7, 9, K=12, R=4, S_open=2, extent=(4.0, 60.0))
    f = optim.Fitter(bz.Rasterizer(sc), optim.FitConfig(optimizer=optimizer, **kw))
    return f


def _gradients(f, seed):
    import torch
    g = torch.Generator().manual_seed(seed)
    for d in (f.rast.d_ctrl, f.rast.d_color, f.rast.d_opacity, f.rast.d_width):
        d.copy_(1e-3 * torch.randn(d.shape, generator=g))
    f.rast.d_color.view(-1)[3] = float("nan")
    f.rast.d_opacity.view(-1)[1] = 0.0


def _state(f):
    out = {}
    for name in ("ctrl_n", "color", "opacity", "width"):
        p = getattr(f, name)
        st = f.opt.state[p]
        out[name] = [t.detach().double().cpu().numpy() for t in
                     (p, st["exp_avg"], st["exp_avg_sq"], p.grad)] + [float(st["step"])]
    return out


@pytest.mark.gpu
def test_update_matches_torch():
    from paper_2503_16424_amd import optim
    a, b = _fitter(**optim.PAPER_LR), _fitter(**optim.PAPER_LR)
    b.opt.register_step_post_hook(lambda *_: None)        # a hooked step is torch's own
    for f in (a, b):                                      # the first makes the state
        _gradients(f, 1)
        f.update()
    for step in range(2, 5):
        used = a._update_in_one_launch
        calls = []
        a._update_in_one_launch = lambda: calls.append(used()) or calls[-1]
        for f in (a, b):
            _gradients(f, step)
            before = f.ctrl_n._version
            f.update()
            assert f.ctrl_n._version > before
        del a._update_in_one_launch
        assert calls == [True]
        x, y = _state(a), _state(b)
        for name, lr in zip(x, (2e-4, 1e-2, 1e-1, 1e-2)):
            (p, m, v, g, t), (q, n, w, h, u) = x[name], y[name]
            assert t == u == step and np.array_equal(g, h, equal_nan=True)
            assert np.array_equal(np.isnan(p), np.isnan(q))
            ok = ~np.isnan(q)
            assert np.all(np.abs(m - n)[ok] <= 1e-6 * (np.abs(n) + np.abs(h))[ok]), name
            assert np.all(np.abs(v - w)[ok] <= 1e-6 * w[ok]), name
            # the steps differ by the bounds above, and the next starts from the last's end
            tol = (step - 1) * (2e-6 * 10 * lr + 2.0 ** -23 * np.maximum(np.abs(q), 1.0))
            assert np.all(np.abs(p - q)[ok] <= tol[ok]), name
        assert np.nanmin(x["width"][0]) >= 0.5 - 1e-7 and np.nanmax(x["opacity"][0]) <= 1.0


@pytest.mark.gpu
def test_push_copies_the_bits():
    import torch
    f = _fitter()
    with torch.no_grad():
        f.ctrl_n.mul_(1.37)
        f.ctrl_n.view(-1)[5] = float("nan")
        f.width.add_(0.123)
        f.color.view(-1)[2] = -0.0
    version = f.rast.ctrl._version
    f.push()
    assert f.rast.ctrl._version > version
    want = (f.ctrl_n.detach() + 1.0) * f.half
    assert torch.equal(f.rast.ctrl.view(torch.int32), want.view(torch.int32).view(f.rast.ctrl.shape))
    assert torch.equal(f.rast.stroke_w, f.width.detach())
    assert torch.equal(f.rast.color.view(torch.int32), f.color.detach().view(torch.int32))
    assert torch.equal(f.rast.opacity, f.opacity.detach())


@pytest.mark.gpu
@pytest.mark.parametrize("case", ["hook", "scheduler", "decay", "amsgrad", "sgd", "moved", "tensor_lr"])
def test_other_optimisers_take_their_own_step(case):
    import torch
    f = _fitter("sgd" if case == "sgd" else "adam")
    calls = []
    if case == "hook":
        f.opt.register_step_pre_hook(lambda *_: calls.append(1) and None)
    elif case == "scheduler":
        torch.optim.lr_scheduler.StepLR(f.opt, 5)
    elif case == "decay":
        f.opt.param_groups[0]["weight_decay"] = 0.1
    elif case == "amsgrad":
        f.opt.param_groups[1]["amsgrad"] = True
    elif case == "tensor_lr":
        f.opt.param_groups[2]["lr"] = torch.tensor(1e-2)
    elif case == "moved":
        f.opt.param_groups[0], f.opt.param_groups[1] = f.opt.param_groups[1], f.opt.param_groups[0]
    for step in range(2):
        _gradients(f, step)
        assert not f._update_in_one_launch()
        f.update()
    assert len(calls) == (2 if case == "hook" else 0)


def test_arguments_are_checked_on_the_host():
    from paper_2503_16424_amd import bz
    lib = bz.load_library()
    one = (bz.AdamGroup * 1)()
    assert lib.bz_adam_step(None, 0, None) == bz.BZ_OK
    assert lib.bz_adam_step(one, 1, None) == bz.BZ_OK                  # empty array
    assert lib.bz_adam_step(None, 1, None) == bz.BZ_ERR_ARG
    assert lib.bz_adam_step(one, -1, None) == bz.BZ_ERR_ARG
    assert lib.bz_adam_step((bz.AdamGroup * 9)(), 9, None) == bz.BZ_ERR_ARG
    one[0].n = 4
    assert lib.bz_adam_step(one, 1, None) == bz.BZ_ERR_ARG             # no arrays
    one[0].n = -1
    assert lib.bz_adam_step(one, 1, None) == bz.BZ_ERR_ARG
    cp = (bz.AffineGroup * 1)()
    assert lib.bz_affine_copy(cp, 1, None) == bz.BZ_OK
    cp[0].n = 4
    assert lib.bz_affine_copy(cp, 1, None) == bz.BZ_ERR_ARG
    cp[0].src = C.c_void_p(4096).value
    assert lib.bz_affine_copy(cp, 1, None) == bz.BZ_ERR_ARG
