"""Distance joins with radii that are subnormal, or whose squares underflow:
the choice of the cells ends, and a point on a centre is its pair."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [0.0, 5e-324, 1e-323, 5e-323, 1e-322, 1e-310, 1e-200])
@pytest.mark.parametrize("centre", [(0.0, 0.0), (1.0, 1.0)])
@pytest.mark.parametrize("n", [3, 5000])
def test_tiny_radii(ctx, n, centre, r):
    x, y = np.full(n, centre[0]), np.full(n, centre[1])
    x[1::3] += 2.0
    y[2::3] -= 2.0
    dx, dy = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    for nd in (1, 4):
        cx, cy = np.full(nd, centre[0]), np.full(nd, centre[1])
        if nd > 1:
            cx[2] += 5.0
        near = [j for j in range(nd) if cx[j] == centre[0]]
        pt, pd = ctx.distance_join(dx, dy, cx, cy, r)
        ids = np.arange(0, n, 3)
        assert np.array_equal(pt.cpu().numpy(), np.repeat(ids, len(near)))
        assert np.array_equal(pd.cpu().numpy(), np.tile(near, ids.size))
        cnt = ctx.distance_join_count(dx, dy, cx, cy, r).cpu().numpy()
        assert np.array_equal(cnt, [ids.size if j in near else 0 for j in range(nd)])
