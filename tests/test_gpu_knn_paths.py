"""kNN at the edges of its paths: candidates from the words that reach the
circle (up to a 32nd of the points) or from a selection over all points, and
ordered by one workgroup (up to 4,096) or by the library sort.  Ids are
decided exactly and equal the oracle's."""
import numpy as np
import pytest
import torch

from oracle import disk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(63, 5), (65, 64), (4096, 4096), (4097, 4097), (40_000, 1), (40_000, 300),
                                 (40_000, 2500), (300_000, 1000), (300_000, 5000)])
@pytest.mark.parametrize("lattice", [False, True])
def test_knn_paths(ctx, n, k, lattice):
    rng = np.random.default_rng(n + k)
    if lattice:   # many equal distances
        side = int(np.ceil(np.sqrt(n)))
        x, y = (a.ravel()[:n].astype(np.float64) for a in np.meshgrid(np.arange(side), np.arange(side)))
        p = rng.permutation(n)
        x, y, q = x[p], y[p], (float(side // 2), float(side // 2))
    else:
        x, y, q = rng.normal(0, 100, n), rng.normal(0, 100, n), (3.25, -7.5)
    x[n // 2], y[n // 3] = np.nan, np.inf
    got = ctx.knn(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), q[0], q[1], k).cpu().numpy()
    assert np.array_equal(got.astype(np.int64), np.asarray(disk.knn(x, y, q[0], q[1], k)).astype(np.int64))
