"""Claimant records of rows where interiors overlap: combs of teeth whose
widths in pixels lie about the limits from which 8 lanes or a wavefront walk a span, at
offsets that shift them across lanes, with rows of fewer and of more entries
than a wavefront and than the staging.  Pairs are whole numbers decided
exactly, compared with the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_14362_amd import Context
from workloads import gen

pytestmark = pytest.mark.gpu
EXTENT = 1024


def _comb(width, gap, shift, top):
    """A base with teeth of `width` every `width + gap`, from y = 0 to `top`."""
    ring = [(0.0, -8.0), (float(EXTENT), -8.0), (float(EXTENT), 0.0)]
    a = np.arange(shift, EXTENT - width - 1, width + gap, dtype=float)[::-1]
    for v in a:
        ring += [(v + width, 0.0), (v + width, top), (v, top), (v, 0.0)]
    return np.asarray(ring + [(0.0, 0.0)])


@pytest.mark.parametrize("width", [1.5, 7, 8, 9, 31, 32, 33, 63, 64, 65, 500])
def test_comb_spans(width):
    rings = [_comb(width, 2.0 + k, 3.0 + k, 20.0 + k) for k in range(5)]
    rings += [np.array([[100.0 + 7 * k, -20.0], [900.0 - 5 * k, -20.0], [900.0 - 5 * k, 30.0], [100.0 + 7 * k, 30.0]])
              for k in range(4)]
    polys, n = gen.polys_from_rings(rings), 20_001
    rng = np.random.default_rng(int(2 * width))
    x, y = rng.uniform(-5, EXTENT + 5, n), rng.uniform(-25, 35, n)
    x[::3] = np.round(x[::3])
    want = [np.asarray(a).astype(np.int64) for a in oracle.join_pairs(x, y, polys)]
    count = np.asarray(oracle.join_count(x, y, polys)).astype(np.int64)
    dx, dy = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    c = Context(0)
    for size in ((EXTENT, 64), (300, 9), (4096, 40)):
        c.set_canvas_size(*size)
        cv = c.canvas(polys)
        got = c.join_pairs(dx, dy, cv)
        assert all(np.array_equal(g.cpu().numpy().astype(np.int64), w) for g, w in zip(got, want)), size
        assert np.array_equal(c.join_count(dx, dy, cv).cpu().numpy().astype(np.int64), count), size
        cv.close()
    c.close()
