"""Points beside the ends of segments much longer than the distance, from 2^20
points on (where the floating-point filter decides first) and below: kept or
not as rational arithmetic says, one by one."""
import numpy as np
import pytest
import torch

from oracle.buffer import seg_within_exact
from workloads import gen

pytestmark = pytest.mark.gpu

UP = 1.0 + 1e-11
ENDS = [((-1e7, 0.0), (0.0, 0.0), (-9e-10, 5e-5), 5e-5 * UP),
        ((-1e10, 0.0), (0.0, 0.0), (-9e-7, 0.1), 0.1 * UP),
        ((-626933.8878006589, -1.3669754518551256), (0.0, 0.0), (2.395740662435006e-11, -9.081319519216338e-08),
         9.081319535221679e-08),
        ((-241033.17544444726, 499993.5385700445), (500000.66551455046, 500000.00723007496),
         (500000.66551455046, 500000.0072300682), 6.752088665941962e-09)]


@pytest.mark.parametrize("n", [1001, (1 << 20) + 1])
@pytest.mark.parametrize("turn", [False, True])
@pytest.mark.parametrize("case", range(len(ENDS)))
def test_ends(ctx, case, turn, n):
    a, b, p, r = ENDS[case]
    rng = np.random.default_rng(case)
    # the point itself and others around both ends
    off = rng.uniform(-1.5 * r, 1.5 * r, (1000, 2))
    pts = np.concatenate([[p], np.asarray(b) + off[:500], np.asarray(a) + off[500:]])
    line = gen.polys_from_rings([[np.array([b, a] if turn else [a, b])]])
    want = np.array([seg_within_exact(*q, *a, *b, r) for q in pts])
    pts, want = np.resize(pts, (n, 2)), np.resize(want, n)
    x, y = (torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in pts.T)
    got = ctx.select_near_lines(x, y, line, r).cpu().numpy().astype(np.int64)
    assert np.array_equal(got, np.flatnonzero(want))
