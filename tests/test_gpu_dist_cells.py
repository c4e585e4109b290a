"""The cells of the distance joins: fine cells that disks hold wholly, cells of
more than 32 disks (walked again by the write pass) and of more than 64 (lists
from a key sort), words with more pairs than the write pass stages, lattice
points on circles on both sides of the filtered count pass (2^20 points), and
a capacity below the result.  Pairs are decided exactly, compared with the
oracle's."""
import numpy as np
import pytest
import torch

from oracle import disk

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _check(ctx, x, y, cx, cy, r):
    pt, pd = ctx.distance_join(_dev(x), _dev(y), cx, cy, r)
    opt, opd = disk.distance_join(x, y, cx, cy, r)
    assert np.array_equal(pt.cpu().numpy().astype(np.int64), opt.astype(np.int64))
    assert np.array_equal(pd.cpu().numpy().astype(np.int64), opd.astype(np.int64))
    cnt = ctx.distance_join_count(_dev(x), _dev(y), cx, cy, r).cpu().numpy().astype(np.int64)
    assert np.array_equal(cnt, np.bincount(opd.astype(np.int64), minlength=len(cx)))


@pytest.mark.parametrize("n", [1, 63, 64, 65, 511, 512, 513, 70_001])
def test_sizes(ctx, n):
    rng = np.random.default_rng(n)
    x, y = rng.uniform(0, 1000, n), rng.uniform(0, 1000, n)
    if n > 10:
        x[3], y[7] = np.nan, np.inf
    cx, cy = rng.uniform(0, 1000, 40), rng.uniform(0, 1000, 40)
    _check(ctx, x, y, cx, cy, 90.0)
    _check(ctx, x, y, cx, cy, rng.uniform(0, 200.0, 40))


@pytest.mark.parametrize("nd", [32, 33, 64, 65, 300])
def test_many_disks_per_cell(ctx, nd):
    """Disks on top of each other: every cell lists up to all of them."""
    rng = np.random.default_rng(nd)
    x, y = rng.uniform(0, 100, 3001), rng.uniform(0, 100, 3001)
    cx, cy = 50 + rng.uniform(-3, 3, nd), 50 + rng.uniform(-3, 3, nd)
    _check(ctx, x, y, cx, cy, rng.uniform(5, 40, nd))


@pytest.mark.parametrize("n", [(1 << 20) - 1, (1 << 20) + 1])
def test_lattice_both_count_passes(ctx, n):
    side = 1 << 10
    k = np.arange(n)
    x, y = (k % side).astype(np.float64), (k // side).astype(np.float64)
    rng = np.random.default_rng(3)
    cx, cy = rng.integers(0, side, 30).astype(np.float64), rng.integers(0, side, 30).astype(np.float64)
    _check(ctx, x, y, cx, cy, 25.0)
    _check(ctx, x, y, cx, cy, np.where(np.arange(30) % 2, 65.0, 5.0))


def test_one_large_disk_and_shifted(ctx):
    rng = np.random.default_rng(9)
    for shift in (0.0, 2.0 ** 32):
        x, y = rng.uniform(0, 1000, 50_000) + shift, rng.uniform(0, 1000, 50_000) - shift
        cx, cy = rng.uniform(0, 1000, 60) + shift, rng.uniform(0, 1000, 60) - shift
        r = np.full(60, 4.0)
        r[7] = 700.0
        _check(ctx, x, y, cx, cy, r)


def test_capacity(ctx):
    rng = np.random.default_rng(11)
    x, y = rng.uniform(0, 100, 20_000), rng.uniform(0, 100, 20_000)
    cx, cy = rng.uniform(0, 100, 50), rng.uniform(0, 100, 50)
    full = ctx.distance_join(_dev(x), _dev(y), cx, cy, 12.0)
    small = ctx.distance_join(_dev(x), _dev(y), cx, cy, 12.0, cap=5)   # retried with the total
    assert all(torch.equal(a, b) for a, b in zip(full, small))
