"""Convolutions on both sides of the dispatch's lines (GPU): filters too large for a block
of 64 output channels with few and with many pixels (16-channel blocks or the general
kernel), and filter gradients whose chunks of pixels are fewer than the XCDs.

Against FP64 sums of the same BF16 operands: every pass accumulates K products in FP32,
so K times 2^-24 of the sum of |terms| bounds it; outputs in BF16 add half a unit in the
last place (2^-9)."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [  # n, h, w, c, k, r, stride, pad
    (61, 8, 8, 128, 128, 3, 1, 1),      # 3,904 pixels: 62 wide blocks
    (259, 8, 8, 128, 128, 3, 1, 1),     # 16,576: 260
    (67, 8, 8, 256, 200, 3, 1, 1),      # 136 forward, 136 back
    (65, 16, 16, 192, 136, 3, 2, 1),    # four classes
    (9, 7, 5, 512, 512, 3, 1, 1),       # filter gradient in one or two chunks
    (40, 9, 11, 384, 520, 1, 1, 0),
    (3, 1, 1, 512, 264, 1, 1, 0),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_passes_match_fp64(shape):
    import torch
    from torch.nn.functional import unfold
    from paper_2503_16424_amd import cnn
    n, h, w, c, k, r, s, p = shape
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    d = cnn.conv_desc(n, h, w, c, k, r, s, p)
    x = torch.randn((n, h, w, c), generator=g, device="cuda").to(torch.bfloat16)
    wt = (torch.randn((k, r, r, c), generator=g, device="cuda") * 0.1).to(torch.bfloat16)
    dy = torch.randn((n, d.ho, d.wo, k), generator=g, device="cuda")
    y = torch.empty((n, d.ho, d.wo, k), device="cuda")
    yb = torch.empty_like(y, dtype=torch.int16)
    dx, dw, db = (torch.empty(t.shape, device="cuda") for t in (x, wt, dy[0, 0, 0]))
    xi, wi = x.view(torch.int16), wt.view(torch.int16)
    cnn.conv_fwd(d, xi, wi, None, relu=False, y=y)
    cnn.conv_fwd(d, xi, wi, None, relu=False, y_bf16=yb)
    cnn.conv_bwd_data(d, dy, wi, dx)
    cnn.conv_bwd_weight(d, dy, xi, dw, db)

    # FP64, as matrix products of patches [n, c r r, pixels]; dy as the kernels round it
    def columns(t):
        return unfold(t.double().permute(0, 3, 1, 2), r, padding=p, stride=s)

    def products(f):
        X, W = f(columns(x)), f(wt.double().permute(0, 3, 1, 2).reshape(k, -1))
        D = f(dy.to(torch.bfloat16).double().reshape(n, -1, k))
        Y = torch.matmul(W, X).permute(0, 2, 1).reshape(y.shape)
        C = torch.matmul(D.reshape(-1, k), W).view(n, -1, c * r * r).permute(0, 2, 1)
        X2 = X.permute(0, 2, 1).reshape(-1, c * r * r)
        G = torch.matmul(D.reshape(-1, k).t().contiguous(), X2)
        back = torch.nn.functional.fold(C, (h, w), r, padding=p, stride=s).permute(0, 2, 3, 1)
        return Y, back, G.view(k, c, r, r).permute(0, 2, 3, 1)

    want, scale = products(lambda t: t), products(torch.abs)
    for got, ref, sc, terms, what in zip((y, dx, dw), want, scale,
                                         (c * r * r, k * r * r, n * d.ho * d.wo),
                                         ("forward", "input", "filter")):
        assert ((got.double() - ref).abs() <= terms * 2.0 ** -24 * sc + 1e-30).all(), what
    assert torch.equal(yb.view(torch.bfloat16), y.to(torch.bfloat16))
    pixels = n * d.ho * d.wo
    flat = dy.double().view(-1, k)
    assert ((db.double() - flat.sum(0)).abs() <= pixels * 2.0 ** -24 * flat.abs().sum(0)).all()
