"""Join pairs over a table with long lists of polygons per point: lengths around
the one from which a list goes through a bitmap, ids in several windows of it,
layered sets (ids in any order) and a capacity inside a list.  Squares around
one centre: a point's list is those whose half side exceeds its distance."""
import ctypes
import time

import numpy as np
import pytest
import torch

from paper_2203_14362_amd import SPADE_E_CAPACITY
from workloads import gen

pytestmark = pytest.mark.gpu


def _squares(half):
    return gen.polys_from_rings([[np.array([[-h, -h], [h, -h], [h, h], [-h, h]])] for h in half])


def _expected(x, y, half):
    inside = np.maximum(np.abs(x), np.abs(y))[:, None] < half[None, :]
    return np.nonzero(inside)


def _pairs(ctx, b, t, cap):
    pt, pg = (torch.full((max(cap, 1),), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    n = ctypes.c_int64()
    rc = ctx.lib.spade_batch_join_pairs(ctx.handle, b.handle, t.handle, ctypes.c_void_p(pt.data_ptr()),
                                        ctypes.c_void_p(pg.data_ptr()), cap, ctypes.byref(n))
    return rc, n.value, pt.cpu().numpy()[:cap].astype(np.int64), pg.cpu().numpy()[:cap].astype(np.int64)


@pytest.mark.parametrize("m,layered", [(m, lay) for m in (47, 48, 49, 55, 130, 300) for lay in (False, True)] + [(2100, False)])
def test_lengths(ctx, m, layered):
    n = 9001
    rng = np.random.default_rng(m)
    half = rng.permutation(np.concatenate([np.full(m - m // 8, 2.0) + np.arange(m - m // 8) * 1e-3,
                                           rng.uniform(0, 1, m // 8)]))
    x, y = rng.uniform(-1, 1, n), rng.uniform(-1, 1, n)
    x[::5] *= 3.0
    polys = _squares(half)
    t = ctx.table(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    b = ctx.layered(polys) if layered else ctx.batch(polys, np.arange(m + 1))
    want = _expected(x, y, half)
    pt, pg = ctx.batch_join_pairs(b, t)
    for got, w in zip((pt, pg), want):
        assert np.array_equal(got.cpu().numpy().astype(np.int64), w)
    for cap in (1, want[0].size // 2, want[0].size - 3):
        rc, total, gp, gg = _pairs(ctx, b, t, cap)
        assert rc == SPADE_E_CAPACITY and total == want[0].size
        assert np.array_equal(gp, want[0][:cap]) and np.array_equal(gg, want[1][:cap])
    b.close()
    t.close()


@pytest.mark.parametrize("far", [70, 200])
def test_ids_in_several_windows(ctx, far):
    """A grid of 70,225 cells between two groups of squares around all of it."""
    side, n = 265, 2001
    rng = np.random.default_rng(far)
    half = side + rng.permutation(np.arange(2 * far)) * 0.5
    grid = gen.rect_grid(side, side, -side / 2, -side / 2, 1.0, 1.0)
    polys = gen.concat_polys(gen.concat_polys(_squares(half[:far]), grid), _squares(half[far:]))
    bound = np.concatenate([np.arange(far + 1), far + side * side + np.arange(far + 1)])
    x, y = rng.uniform(-side / 2, side / 2, n), rng.uniform(-side / 2, side / 2, n)
    t = ctx.table(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    b = ctx.batch(polys, bound)
    pt, pg = (v.cpu().numpy().astype(np.int64) for v in ctx.batch_join_pairs(b, t))
    cell = far + np.floor(y + side / 2).astype(np.int64) * side + np.floor(x + side / 2).astype(np.int64)
    want = np.concatenate([np.broadcast_to(np.arange(far), (n, far)), cell[:, None],
                           np.broadcast_to(far + side * side + np.arange(far), (n, far))], axis=1)
    assert np.array_equal(pt, np.repeat(np.arange(n), 2 * far + 1))
    assert np.array_equal(pg, want.ravel())
    b.close()
    t.close()


def test_time_grows_with_the_list(ctx):
    """By insertion 2,000 polygons over each of 30,000 points took seconds."""
    m, n = 2000, 30_000
    half = 2.0 + np.random.default_rng(1).permutation(m) * 1e-3
    p = torch.rand(n, device="cuda", dtype=torch.float64)
    t = ctx.table(p, p.flip(0).contiguous())
    b = ctx.batch(_squares(half), np.arange(m + 1))
    ctx.batch_join_pairs(b, t)
    torch.cuda.synchronize()
    a = time.perf_counter()
    pt, pg = ctx.batch_join_pairs(b, t)
    torch.cuda.synchronize()
    assert time.perf_counter() - a < 0.5
    assert torch.equal(pg.view(n, m), torch.arange(m, device="cuda", dtype=torch.int32).expand(n, m))
    assert torch.equal(pt.view(n, m)[:, 0], torch.arange(n, device="cuda", dtype=torch.int32))
    b.close()
    t.close()
