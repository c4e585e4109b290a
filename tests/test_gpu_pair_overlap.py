"""Whether the pairs' count pass keeps labels follows the pixels inside several
polygons: tessellations of any resolution, polygons whose interiors share
pixels, and polygons that overlap in boundary pixels alone (found by the count
pass).  Through a resident canvas and through the plain call.  Pairs are whole
numbers decided exactly, compared with the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_14362_amd import Context
from workloads import gen

pytestmark = pytest.mark.gpu


def _sets():
    yield "tessellation", gen.rect_grid(12, 9, 0.0, 0.0, 1.0, 1.0)
    yield "overlapping", gen.concat_polys(gen.rect_grid(12, 9, 0.0, 0.0, 1.0, 1.0),
                                          gen.star_polygon(60, 0.1, (6.0, 4.5), L=9.0, seed=4))
    rng = np.random.default_rng(3)
    c = rng.uniform(0.2, 8.8, (300, 2))
    tri = np.array([[-0.15, -0.1], [0.15, -0.1], [0.0, 0.2]])
    yield "small", gen.polys_from_rings([[p + tri] for p in c])


SETS = dict(_sets())


@pytest.mark.parametrize("size", [(1, 1), (5, 3), (64, 64), (1000, 700)])
@pytest.mark.parametrize("name", sorted(SETS))
def test_pairs(name, size):
    polys, n = SETS[name], 30_001
    rng = np.random.default_rng(n)
    x, y = rng.uniform(-1, 13, n), rng.uniform(-1, 10, n)
    x[::13], y[::11] = np.round(x[::13]), np.round(y[::11])
    want = [np.asarray(a).astype(np.int64) for a in oracle.join_pairs(x, y, polys)]
    dx, dy = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    c = Context(0)
    c.set_canvas_size(*size)
    cv = c.canvas(polys)
    for target in (cv, polys, c.polys(polys), polys):   # the first plain call grows the canvas
        got = c.join_pairs(dx, dy, target)
        assert all(np.array_equal(g.cpu().numpy().astype(np.int64), w) for g, w in zip(got, want))
    cv.close()
    c.close()
