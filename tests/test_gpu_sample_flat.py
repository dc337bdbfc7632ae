"""Short curves share a wave in the sampler (GPU): records and tile lists of curve
sets on both sides of the 64-Gaussian line, where curves and waves end differently.

The records must be those the reference computes in FP64, to the tolerances of the
sampler's own test; the two calls and the combined one must give the same bits, and a
set whose longest curve moves it to the other kernel the same records up to the last
bit of FP32 (both evaluate in FP64, in their own order).
"""
import numpy as np
import pytest

from paper_2503_16424_amd import scenes
from tests.helpers import sample_bin_matches_separate

pytestmark = pytest.mark.gpu


def _scene(name):
    if name == "one":
        return scenes.uniform_open(1, 64, 64, 1, 2)
    if name == "two_samples":                     # 32 curves per wave and a remainder
        return scenes.uniform_open(2, 100, 80, 333, 2)
    if name == "K63":                             # every curve straddles two waves
        return scenes.uniform_open(3, 200, 100, 70, 63, S=2)
    if name == "K64":
        return scenes.uniform_open(4, 200, 100, 65, 64, S=3, per_segment_opacity=True)
    if name == "closed":
        return scenes.mixed(5, 160, 120, 40, 60, K=8, R=6, S_open=2, extent=(4.0, 60.0))
    if name == "many":                            # more than 64^2 curves
        return scenes.uniform_open(6, 512, 512, 5000, 5)
    return [scenes.uniform_open(7 + i, 60 + 30 * i, 50, 20 * i + 1, 9) for i in range(4)]


@pytest.mark.parametrize("radix", [False, True])
@pytest.mark.parametrize("name", ["one", "two_samples", "K63", "K64", "closed", "many", "batch"])
def test_flat_sampling_matches_the_per_curve_kernel(name, radix):
    import torch
    from paper_2503_16424_amd import bz
    sc = _scene(name)
    r = bz.Rasterizer(sc, bz.RenderOptions(radix_bins=radix))
    assert r.curves.max_gauss_per_curve <= 64
    r.render()
    sample_bin_matches_separate(torch, r)
    rec = r.rec[: 12 * r.n_gauss].clone()
    pairs = r.pairs_required()
    r.curves.max_gauss_per_curve = 65             # an upper bound: the other kernel
    r.sample_bin()
    other = r.rec[: 12 * r.n_gauss]
    a, b = rec.view(-1, 12).double().cpu().numpy(), other.view(-1, 12).double().cpu().numpy()
    assert np.array_equal(rec.view(-1, 12)[:, 8:].view(torch.int32).cpu(),
                          other.view(-1, 12)[:, 8:].view(torch.int32).cpu())
    # mean (hi + lo): FP64 to 2^-47 of the canvas; shape: one rounding to FP32
    assert np.abs((a[:, :2] + a[:, 2:4]) - (b[:, :2] + b[:, 2:4])).max() <= 1e-9
    assert np.all(np.abs(a[:, 4:8] - b[:, 4:8]) <= 2.0 ** -22 * np.abs(b[:, 4:8]).max(1, keepdims=True))
    assert abs(r.pairs_required() - pairs) <= max(2, pairs // 1000)
