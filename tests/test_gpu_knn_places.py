"""kNN around places that hold many points: tens of thousands of equal distances
among more candidates than one workgroup orders and fewer than a 128th of the
points, so that they are taken from the words that reach the circle and ordered
by the library sort.  The ids are exact and equal the oracle's, in its order;
the time of a call shows work that grows with the square of a place."""
import time

import numpy as np
import pytest
import torch

from oracle import disk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("at", [(0.0, 0.0), (3.0, 4.0)])   # the query point itself, five units off
def test_crowded_place(ctx, at):
    n, many, k = 5_300_001, 30_000, 39_000
    rng = np.random.default_rng(11)
    x, y = rng.uniform(100, 200, n), rng.uniform(100, 200, n)
    place = rng.permutation(n)[:40_000]
    x[place[:many]], y[place[:many]] = at
    # four more places at one distance, and points around them (all within the
    # circle of radius 8)
    for j, (a, b) in enumerate([(6.0, 0.0), (0.0, 6.0), (-6.0, 0.0), (0.0, -6.0)]):
        p = place[many + 1500 * j:many + 1500 * (j + 1)]
        x[p], y[p] = a, b
    rest = place[many + 6000:]
    x[rest], y[rest] = rng.uniform(-5.6, 5.6, rest.size), rng.uniform(-5.6, 5.6, rest.size)
    dx, dy = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    torch.cuda.synchronize()
    t = time.perf_counter()
    got = ctx.knn(dx, dy, 0.0, 0.0, k).cpu().numpy()
    assert time.perf_counter() - t < 5.0
    assert np.array_equal(got.astype(np.int64), np.asarray(disk.knn(x, y, 0.0, 0.0, k)).astype(np.int64))
