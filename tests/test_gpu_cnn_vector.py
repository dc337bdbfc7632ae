"""Vector form of the convolutions at the edges of its tiles (GPU).

Channel counts that are multiples of 8 and aligned operands take the vector
kernels; the same operands 8 bytes off alignment take the general ones.  Forward
and input gradient add the same products in the same order, so the two must give
the same bits, whatever the values.  The filter and bias gradients differ by the
FP32 accumulation order only: 1e-5 of the sum of |terms| against FP64.
"""
import numpy as np
import pytest

from oracle import cnn_oracle as co

pytestmark = pytest.mark.gpu

SHAPES = [  # n, h, w, c, k, r, stride, pad
    (7, 61, 59, 8, 68, 3, 1, 1),      # 64 and 4 channels per block, k = 72 of 96
    (6, 131, 127, 24, 72, 1, 2, 0),   # blocks of all four classes, three without a tap
    (6, 131, 127, 16, 64, 3, 2, 1),   # the same, classes of 1, 2, 2 and 4 taps
    (6, 65, 67, 16, 24, 3, 2, 1),     # a class per workgroup
    (2, 20, 21, 16, 8, 3, 4, 1),      # sixteen classes, seven of them without a tap
    (3, 9, 7, 72, 40, 3, 1, 1),       # 16 channels per workgroup, N = 8 of 16 in the last
    (1, 1, 1, 8, 8, 1, 1, 0),         # one pixel
    (2, 5, 4, 480, 8, 3, 1, 1),       # filters of 16 channels do not fit: the general kernel
]


def _shifted(torch, t):
    """A copy of t whose storage starts 8 bytes past a 16-byte boundary."""
    off = 8 // t.element_size()
    buf = torch.empty(t.numel() + off, dtype=t.dtype, device=t.device)
    out = buf[off:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_vector_form_equals_the_general_one(shape, special):
    import torch
    from paper_2503_16424_amd import cnn
    n, h, w, c, k, r, s, p = shape
    g = torch.Generator().manual_seed(sum(shape))
    d = cnn.conv_desc(n, h, w, c, k, r, s, p)

    def bf16(*size):
        return torch.randn(size, generator=g).to(torch.bfloat16)

    x, wt, dy = bf16(n, h, w, c), bf16(k, r, r, c) * 0.2, torch.randn((n, d.ho, d.wo, k), generator=g)
    bias = torch.randn(k, generator=g)
    if special:
        x.view(-1)[::97] = float("inf")
        x.view(-1)[5::89] = float("nan")
        dy.view(-1)[::101] = float("-inf")
        dy.view(-1)[7::103] = float("nan")
    xg, wg = x.view(torch.int16).cuda(), wt.view(torch.int16).cuda()
    dyg, bg = dy.cuda(), bias.cuda()

    def run(xg, wg, dyg, off):
        like = (lambda t: _shifted(torch, t)) if off else (lambda t: t)
        y = like(torch.zeros((n, d.ho, d.wo, k), device="cuda"))
        yb = like(torch.zeros((n, d.ho, d.wo, k), dtype=torch.int16, device="cuda"))
        dx = like(torch.zeros((n, h, w, c), device="cuda"))
        dw, db = torch.empty((k, r, r, c), device="cuda"), torch.empty(k, device="cuda")
        cnn.conv_fwd(d, xg, wg, bg, relu=False, y=y)
        cnn.conv_fwd(d, xg, wg, bg, relu=True, y_bf16=yb)
        cnn.conv_bwd_data(d, dyg, wg, dx, x_mask=xg)
        cnn.conv_bwd_weight(d, dyg, xg, dw, db)
        return [t.cpu() for t in (y, yb, dx, dw, db)]

    fast = run(xg, wg, dyg, False)
    slow = run(*(_shifted(torch, t) for t in (xg, wg, dyg)), True)
    for a, b in zip(fast[:3], slow[:3]):
        if a.dtype == torch.int16:
            a, b = a.view(torch.bfloat16), b.view(torch.bfloat16)
        a, b = a.float().numpy(), b.float().numpy()
        assert np.array_equal(a, b, equal_nan=True)
    if special:
        for a, b in zip(fast[3:], slow[3:]):
            assert torch.equal(a.isnan(), b.isnan())
        return
    x64, dyb = x.double().numpy(), co.bf16(dy.numpy())
    ref, _ = co.conv_bwd_weight(dyb, x64, r, s, p)
    scale, _ = co.conv_bwd_weight(np.abs(dyb), np.abs(x64), r, s, p)
    assert (np.abs(fast[3].numpy() - ref) / (scale + 1e-30)).max() <= 1e-5
    d64 = dy.double().numpy().reshape(-1, k)
    assert (np.abs(fast[4].numpy() - d64.sum(0)) / np.abs(d64).sum(0)).max() <= 1e-5


@pytest.mark.parametrize("side,offset", [(32, 0), (32, 1), (16, 0), (5, 0), (33, 0), (1, 0), (4, 2)])
def test_patches_of_every_side(side, offset):
    """Four pixels at a time (side a multiple of 4, aligned output) and one at a time."""
    import torch
    from paper_2503_16424_amd import cnn
    g = torch.Generator().manual_seed(side)
    img = torch.rand((3, 41, 67), generator=g)
    img[0, 3, 4], img[2, 7, 9] = float("inf"), float("nan")
    xy = torch.tensor([[0, 0], [60, 35], [-3, -2], [-100, 5], [33, 20], [66, 40]], dtype=torch.int32)
    n = xy.shape[0]
    buf = torch.empty(n * side * side * 3 + offset, dtype=torch.int16, device="cuda")
    out = buf[offset:].view(n, side, side, 3)
    cnn.extract_patches(img.cuda(), xy.cuda(), side, 0.25, out)
    pad = torch.full((3, 41 + 300, 67 + 300), 0.25)
    pad[:, 150:191, 150:217] = img
    want = torch.stack([pad[:, y + 150: y + 150 + side, x + 150: x + 150 + side].permute(1, 2, 0)
                        for x, y in xy.tolist()]).to(torch.bfloat16)
    assert torch.equal(out.cpu(), want.view(torch.int16)) or torch.equal(
        out.cpu().view(torch.bfloat16).nan_to_num(7.0), want.nan_to_num(7.0))


@pytest.mark.parametrize("shape", [(2, 5, 7, 3), (1, 1, 1, 1), (3, 4, 8), (600, 3)])
def test_channel_padding(shape):
    import torch
    from paper_2503_16424_amd import cnn
    x = torch.randint(-2 ** 15, 2 ** 15, shape, dtype=torch.int16)
    want = torch.nn.functional.pad(x, (0, 8 - shape[-1]))
    assert torch.equal(cnn.pad_channels(x.cuda(), 8).cpu(), want)
    strided = torch.stack([x, x], 0).cuda()[0]
    assert torch.equal(cnn.pad_channels(strided, 8).cpu(), want)


def test_added_filter_gradients():
    import torch
    from paper_2503_16424_amd import cnn
    for n, h, c, k, r, s, p in ((2, 9, 16, 24, 3, 2, 1), (2, 32, 3, 64, 3, 1, 1), (3, 6, 5, 7, 3, 1, 1)):
        d = cnn.conv_desc(n, h, 32 if c == 3 else h, c, k, r, s, p)
        g = torch.Generator(device="cuda").manual_seed(c)
        x = torch.randn((n, d.h, d.w, c), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
        dy = torch.randn((n, d.ho, d.wo, k), generator=g, device="cuda")
        dw, db = torch.empty((k, r, r, c), device="cuda"), torch.empty(k, device="cuda")
        cnn.conv_bwd_weight(d, dy, x, dw, db)
        aw, ab = torch.full_like(dw, 2.0), torch.full_like(db, -3.0)
        cnn.conv_bwd_weight_add(d, dy, x, aw, ab)
        assert ((aw - 2.0) - dw).abs().max() <= 1e-5 * (dw.abs().max() + 2.0)
        assert ((ab + 3.0) - db).abs().max() <= 1e-5 * (db.abs().max() + 3.0)


def _decode_reference(z):
    import torch
    from paper_2503_16424_amd import cnn
    s = torch.sigmoid(z.view(-1, cnn.CURVES, cnn.PER_CURVE))
    return torch.cat([s[..., :8] * (1.0 + 2.0 * cnn.MARGIN) - cnn.MARGIN, s[..., 8:]], dim=-1)


@pytest.mark.parametrize("n", [1, 3, 1024])
def test_decode_without_gradients(n):
    """Sigmoid in FP32 and two roundings: 1e-6 absolute of values up to 1.25."""
    import torch
    from paper_2503_16424_amd import cnn
    g = torch.Generator(device="cuda").manual_seed(n)
    z = torch.randn((n, cnn.OUT), generator=g, device="cuda") * 4
    z.view(-1)[3], z.view(-1)[11], z.view(-1)[5] = float("inf"), float("-inf"), float("nan")
    got, want = cnn.decode(z), _decode_reference(z.double())
    assert got.shape == want.shape and got.dtype == torch.float32
    assert torch.equal(got.isnan(), want.isnan())
    assert (got.double() - want).nan_to_num(0.0).abs().max() <= 1e-6


def test_decode_where_torch_follows():
    import torch
    from paper_2503_16424_amd import cnn
    z = torch.randn((4, cnn.OUT), device="cuda")
    a = z.clone().requires_grad_()
    cnn.decode(a).sum().backward()
    b = z.clone().requires_grad_()
    _decode_reference(b).sum().backward()
    assert torch.equal(a.grad, b.grad)
    t = torch.randn_like(z)
    _, jvp = torch.func.jvp(cnn.decode, (z,), (t,))
    _, ref = torch.func.jvp(_decode_reference, (z,), (t,))
    assert torch.equal(jvp, ref)
    with torch.autograd.forward_ad.dual_level():
        out = cnn.decode(torch.autograd.forward_ad.make_dual(z, t))
        assert torch.equal(torch.autograd.forward_ad.unpack_dual(out).tangent, ref)
    assert torch.equal(torch.func.vmap(cnn.decode)(z.view(4, 1, -1)),
                       torch.func.vmap(_decode_reference)(z.view(4, 1, -1)))
