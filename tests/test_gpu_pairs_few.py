"""Join pairs over a table that is large beside the chunks its queries meet:
sorted keys, and lists where the keys' room does not hold the pairs (several
polygons of a query over each point), at both sides of the rule.  Pairs are
whole numbers decided exactly, compared with the oracle's on the points near
the queries."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2203_14362_amd import SPADE_E_CAPACITY
from workloads import gen

pytestmark = pytest.mark.gpu


def _stars(k, centre, size, seed):
    rng = np.random.default_rng(seed)
    rings = []
    for _ in range(k):
        th = np.linspace(0, 2 * np.pi, 24)[:-1]
        r = size * (1 + 0.3 * rng.uniform(-1, 1, th.size))
        rings.append([np.stack([centre[0] + r * np.cos(th), centre[1] + r * np.sin(th)], 1)])
    return gen.polys_from_rings(rings)


@pytest.mark.parametrize("n", [300_000, (1 << 23) - 1, 1 << 23])
@pytest.mark.parametrize("size", [1e-4, 0.01, 0.05, 0.3])
@pytest.mark.parametrize("shape", ["one", "four queries", "stacked in one query", "layered", "nothing"])
def test_pairs(ctx, n, size, shape):
    g = torch.Generator(device="cuda").manual_seed(n)
    x, y = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) for _ in range(2))
    k = {"one": 1, "four queries": 4, "stacked in one query": 9, "layered": 3, "nothing": 2}[shape]
    centre = (0.4, 0.6) if shape != "nothing" else (5.0, 5.0)
    polys = _stars(k, centre, size, 3)
    t = ctx.table(x, y)
    if shape == "layered":
        b = ctx.layered(polys)
    else:
        b = ctx.batch(polys, [0, k] if shape == "stacked in one query" else np.arange(k + 1))
    near = ((x - centre[0]).abs().maximum((y - centre[1]).abs()) <= 1.4 * size).nonzero().squeeze(1).cpu().numpy()
    wp, wg = oracle.join_pairs(x.cpu().numpy()[near], y.cpu().numpy()[near], polys)
    want = [near[np.asarray(wp).astype(np.int64)], np.asarray(wg).astype(np.int64)]
    pt, pg = ctx.batch_join_pairs(b, t)
    for got, w in zip((pt, pg), want):
        assert np.array_equal(got.cpu().numpy().astype(np.int64), w)
    total = want[0].size
    for cap in sorted({0, 1, total // 2, total}):
        op, og = (torch.full((max(cap, 1) + 1,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        m = ctypes.c_int64()
        rc = ctx.lib.spade_batch_join_pairs(ctx.handle, b.handle, t.handle, ctypes.c_void_p(op.data_ptr()),
                                            ctypes.c_void_p(og.data_ptr()), cap, ctypes.byref(m))
        assert m.value == total and rc == (SPADE_E_CAPACITY if total > cap else 0)
        w = min(cap, total)
        assert torch.equal(op[:w], pt[:w]) and torch.equal(og[:w], pg[:w])
        assert (op[w:] == -7).all() and (og[w:] == -7).all()
    b.close()
    t.close()
