"""A count that is only queued keeps its scratch: calls on other streams of the
same context run behind it.  Above 8,192 polygons the count leaves labels there
that its later kernels read.  Counts are whole numbers: equal, no tolerance."""
import numpy as np
import pytest
import torch

from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", [40, 100])   # the LDS histogram, 16-bit labels
def test_calls_on_another_stream(ctx, side):
    n = 20_000_001
    g = torch.Generator(device="cuda").manual_seed(side)
    x, y = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * side for _ in range(2))
    cv = ctx.canvas(gen.rect_grid(side, side, 0.0, 0.0, 1.0, 1.0))
    star = ctx.canvas(gen.star_polygon(40, 0.3, (side / 2, side / 2), L=float(side), seed=5))
    cell = (y.floor() * side + x.floor()).long()
    want = torch.bincount(cell, minlength=side * side)
    ids = ctx.select(x, y, star)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    out = [torch.empty(side * side, dtype=torch.int64, device="cuda") for _ in range(3)]
    torch.cuda.synchronize()
    for o in out:
        with torch.cuda.stream(a):
            ctx.join_count(x, y, cv, out=o, sync=False)
        with torch.cuda.stream(b):   # its result bits lie where the labels lay
            got = ctx.select(x, y, star)
        assert torch.equal(got, ids)
        with torch.cuda.stream(a):
            ctx.join_count(x, y, cv, out=o, sync=False)
        with torch.cuda.stream(b):
            ctx.knn(x, y, side / 2, side / 2, 50)
    torch.cuda.synchronize()
    for o in out:
        assert torch.equal(o, want)
    cv.close()
    star.close()
