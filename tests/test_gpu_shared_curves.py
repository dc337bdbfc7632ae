"""Stage 2 of the backward with several short curves per wave (GPU): against the form
of one curve per wave, on the same stage-1 gradients.

Sums of at most 64 terms in FP32 in another order: 1e-5 of the largest gradient of the
same kind, per curve set.  The copied planes must be equal.
"""
import numpy as np
import pytest

from paper_2503_16424_amd import scenes

pytestmark = pytest.mark.gpu


def _scene(name):
    if name == "K16":                             # four to a wave, one left over
        return scenes.uniform_open(3, 256, 256, 4097, 16, S=2, per_segment_opacity=True)
    if name == "K9":
        return scenes.uniform_open(4, 256, 256, 4099, 9)
    if name == "K32":
        return scenes.uniform_open(5, 256, 256, 4096, 32, S=4)
    if name == "closed":                          # rows across the lanes of a half wave
        return scenes.mixed(6, 256, 256, 2100, 2100, K=8, R=2, S_open=3, extent=(4.0, 40.0))
    return [scenes.uniform_open(7 + i, 64, 64, 1400 + i, 5 + 9 * i) for i in range(3)]


@pytest.mark.parametrize("name", ["K16", "K9", "K32", "closed", "batch"])
def test_shared_waves_match_a_wave_per_curve(name):
    import torch
    from paper_2503_16424_amd import bz
    r = bz.Rasterizer(_scene(name))
    assert r.curves.max_gauss_per_curve <= 32 and r.curves.n_curves >= 4096
    r.render()
    gen = torch.Generator(device="cuda").manual_seed(1)
    r.d_image.copy_(torch.randn(r.d_image.shape, generator=gen, device="cuda"))
    r.backward()
    planes = r.d_gauss.clone()
    outs = ("d_ctrl", "d_width", "d_color", "d_opacity")
    packed = [getattr(r, k).clone() for k in outs]
    r.backward_curves()                           # from the planes, still shared
    shared = [getattr(r, k).clone() for k in outs]
    assert torch.equal(r.d_gauss, planes)
    longest = r.curves.max_gauss_per_curve
    r.curves.max_gauss_per_curve = 33             # an upper bound: a wave per curve
    r.backward_curves()
    for k, a, b in zip(outs, packed, shared):
        ref = getattr(r, k).double().cpu().numpy()
        scale = np.abs(ref).max()
        assert scale > 0 and longest <= 32
        for t in (a, b):
            assert np.abs(t.double().cpu().numpy() - ref).max() <= 1e-5 * scale, k
