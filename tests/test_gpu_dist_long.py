"""Distance joins whose cells list many disks: lists ordered by one lane (16), by a
wavefront (256), by a workgroup (2,048) and through sorted keys, beside cells
of few disks, and cells of up to 32 with and without disks that hold them.
Pairs are decided exactly, compared with the oracle's."""
import numpy as np
import pytest
import torch

from oracle import disk

pytestmark = pytest.mark.gpu


def _check(ctx, x, y, cx, cy, r):
    dx, dy = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    pt, pd = ctx.distance_join(dx, dy, cx, cy, r)
    opt, opd = disk.distance_join(x, y, cx, cy, r)
    assert np.array_equal(pt.cpu().numpy().astype(np.int64), opt.astype(np.int64))
    assert np.array_equal(pd.cpu().numpy().astype(np.int64), opd.astype(np.int64))
    cnt = ctx.distance_join_count(dx, dy, cx, cy, r).cpu().numpy().astype(np.int64)
    assert np.array_equal(cnt, np.bincount(opd.astype(np.int64), minlength=len(cx)))


@pytest.mark.parametrize("nd", [15, 16, 17, 31, 32, 33, 64, 255, 256, 257, 2047, 2048, 2049, 2300])
@pytest.mark.parametrize("n", [700, 40_001])
def test_long_lists(ctx, nd, n):
    rng = np.random.default_rng(nd)
    x, y = rng.uniform(0, 100, n), rng.uniform(0, 100, n)
    x[:50], y[:50] = 40 + rng.integers(0, 5, 50), 40 + rng.integers(0, 5, 50)
    # nd disks on one spot, and 40 spread ones of the same order
    cx = np.concatenate([50 + rng.uniform(-1e-3, 1e-3, nd), rng.uniform(0, 100, 40)])
    cy = np.concatenate([50 + rng.uniform(-1e-3, 1e-3, nd), rng.uniform(0, 100, 40)])
    p = rng.permutation(nd + 40)
    _check(ctx, x, y, cx[p], cy[p], 6.0)
    if nd < 100:
        _check(ctx, x, y, cx[p], cy[p], rng.uniform(0.5, 30.0, nd + 40))
