"""Tile lists of frames whose pairs lie mostly in one bucket of 256 tiles (GPU): buckets
of more than 256 radix blocks of 4,096 pairs are scanned in parts by several workgroups.
The radix path's lists are the reference; all whole numbers, compared exactly."""
import numpy as np
import pytest

from paper_2503_16424_amd import bz, scenes

pytestmark = pytest.mark.gpu


def _crowded(n, K, rows, W=2048, H=256, faint=50):
    """n strokes inside pixel rows [rows) and a few all over the canvas."""
    rng = np.random.default_rng(n + K)
    ctrl = rng.uniform(0, 1, (n, 1, 2)) * [W, rows[1] - rows[0]] + [0, rows[0]]
    ctrl = ctrl + rng.uniform(-40, 40, (n, 4, 2))
    ctrl[..., 1] = np.clip(ctrl[..., 1], *rows)
    ctrl[:faint] = rng.uniform(0, 1, (faint, 4, 2)) * [W, H]
    return scenes.open_curves(W, H, ctrl, rng.uniform(2, 6, n), rng.uniform(0, 1, (n, 3)),
                              rng.uniform(0.1, 1, n), K)


@pytest.mark.parametrize("n,K,rows,long", [
    (2000, 24, (2, 30), 0),            # no long bucket, a buffer that could hold one
    (14000, 24, (2, 30), 0),           # some 240 blocks
    (15500, 24, (2, 30), 1),           # just over 256
    (50000, 32, (2, 30), 1),           # several supers
    (60000, 32, (2, 62), 2),           # two long buckets
    (150000, 32, (34, 62), 3),         # 13 supers between two buckets of two
])
def test_lists_equal_the_radix_path(n, K, rows, long):
    import torch
    sc = _crowded(n, K, rows)
    got = {}
    for radix in (True, False):
        r = bz.Rasterizer(sc, bz.RenderOptions(radix_bins=radix))
        for _ in range(2):                       # the sums are cleared every time
            r.sample_bin()
        if r.ensure_capacity():
            r.sample_bin()
        pairs = r.pairs_required()
        assert not r.flags() & bz.STATUS_OVERFLOW
        got[radix] = (r.ranges.clone(), r.ids[:pairs].clone())
    assert torch.equal(got[True][0], got[False][0])
    assert torch.equal(got[True][1], got[False][1])
    ranges = got[True][0].view(-1, 2).cpu().numpy().astype(np.int64)
    per = (ranges[:, 1] - ranges[:, 0]).reshape(-1, 256).sum(1)
    assert (per > 256 * 4096).sum() == long, per


@pytest.mark.parametrize("extra", [0, 1])
def test_buffers_where_buckets_may_become_long(extra):
    import torch
    sc = _crowded(3000, 24, (2, 30))
    r = bz.Rasterizer(sc)
    r._alloc_pairs(256 * 4096 + extra)
    r.ids.fill_(-1)
    r.sample_bin()
    ref = bz.Rasterizer(sc, bz.RenderOptions(radix_bins=True))
    ref.sample_bin()
    n = ref.pairs_required()
    assert torch.equal(r.ranges, ref.ranges) and torch.equal(r.ids[:n], ref.ids[:n])
    r._alloc_pairs(n - 1)                        # too small by one: no lists at all
    r.ranges.fill_(-1)
    r.sample_bin()
    assert r.flags() & bz.STATUS_OVERFLOW and not r.ranges.any()
