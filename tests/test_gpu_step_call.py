"""bz_step against its three parts.

Images, blend state, lists and the loss gradient are the same operations: equal bits.
Gradients and the loss differ by the order of float atomics only: 1e-5 of their norm.
"""
import ctypes as C

import pytest

from paper_2503_16424_amd import scenes


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["open", "mixed", "radix", "recompute", "batch", "area", "many",
                                  "persistent", "unaligned"])
def test_step_equals_its_parts(form):
    import torch
    from paper_2503_16424_amd import bz
    opts, kw = bz.RenderOptions(), {}
    sc = scenes.mixed(5, 200, 168, 20, 30, K=16, R=8, S_open=3, extent=(4.0, 120.0))
    if form == "open":
        sc = scenes.uniform_open(3, 130, 70, 100, 16)
    elif form == "radix":
        opts = bz.RenderOptions(radix_bins=True)
    elif form == "persistent":
        opts = bz.RenderOptions(persistent=True)
    elif form == "recompute":
        kw = dict(blend_state="recompute")
    elif form == "batch":
        sc = scenes.batched(3, n_canvas=4, side=(40, 120), curves=(10, 60))
    elif form == "area":
        kw = dict(draw_order="area")
    elif form in ("many", "unaligned"):           # sums past the joint clear
        sc = scenes.uniform_open(4, 256, 256, 8200, 128)
    r = bz.Rasterizer(sc, opts, **kw)
    r.render()
    if form == "unaligned":                       # the scratch needs 4-byte alignment only
        r.bwd_scratch = torch.empty(r.bwd_scratch.numel() + 4, dtype=torch.uint8, device="cuda")[4:]
    n = 3 * r.n_pixels
    tgt = torch.rand(r.image.shape, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    outs = ("image", "d_image", "ranges")
    grads = ("d_ctrl", "d_width", "d_color", "d_opacity", "loss")
    r.sample_bin()
    r.forward_l2(tgt)
    r.backward()
    want = {k: getattr(r, k).clone() for k in outs + grads}
    ids = r.ids[: r.pairs_required()].clone()
    for k in outs + grads:
        getattr(r, k).fill_(7)
    r.bwd_scratch.fill_(0x40)
    r.status.fill_(3)
    r.step(tgt)
    for k in outs:
        assert torch.equal(getattr(r, k).view(torch.int32), want[k].view(torch.int32)), k
    assert torch.equal(r.ids[: r.pairs_required()], ids) and n > 0
    for k in grads:
        d = (getattr(r, k).double() - want[k].double()).norm() / want[k].double().norm()
        assert d <= 1e-5, (k, float(d))


def test_step_checks_its_arguments_on_host():
    from paper_2503_16424_amd import bz
    from tests.test_abi_host import _fake_bins, _fake_curves, _opts
    lib = bz.load_library()
    gr = bz.Grads(4096, 4096, 4096, 4096, 4096)

    def call(c=True, image=8192, target=12288, d_image=16384, scale=0.5, scratch=65536,
             nbytes=16 * 36, grads=gr, cap=16):
        cv, o, g, b = _fake_curves(), _opts(), bz.Gaussians(cap, 0, 4096), _fake_bins()
        return lib.bz_step(C.byref(cv) if c else None, C.byref(o), C.byref(g), C.byref(b), image,
                           None, target, C.c_float(scale), d_image, None, C.byref(grads), scratch,
                           nbytes, None)
    assert call(c=False) == bz.BZ_ERR_ARG
    assert call(image=None) == bz.BZ_ERR_ARG
    assert call(target=None) == bz.BZ_ERR_ARG
    assert call(d_image=8192) == bz.BZ_ERR_ARG                 # the image itself
    assert call(scale=float("nan")) == bz.BZ_ERR_ARG
    assert call(scratch=None) == bz.BZ_ERR_ARG
    assert call(nbytes=16 * 36 - 1) == bz.BZ_ERR_CAPACITY
    assert call(cap=8) == bz.BZ_ERR_CAPACITY
    assert call(grads=bz.Grads(4096, 4096, 4096, 4096, None)) == bz.BZ_ERR_ARG
