"""Pairs over a canvas of several polygons, written from the count pass's
labels: sizes around a word (64 points), a group of eight words and a segment,
polygons that overlap (points are probed again), 16- and 32-bit labels and a
capacity below the result.  Results are whole numbers decided exactly,
compared with the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from workloads import gen

pytestmark = pytest.mark.gpu


def _points(n, w, h, seed):
    rng = np.random.default_rng(seed)
    x, y = rng.uniform(-1, w + 1, n), rng.uniform(-1, h + 1, n)
    x[::13], y[::11] = np.round(x[::13]), np.round(y[::11])   # on cell sides
    if n > 10:
        x[3], y[5] = np.nan, np.inf
    return x, y


def _check(ctx, x, y, polys):
    want_pt, want_poly = oracle.join_pairs(x, y, polys)
    pt, poly = ctx.join_pairs(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), polys)
    assert np.array_equal(pt.cpu().numpy().astype(np.int64), np.asarray(want_pt).astype(np.int64))
    assert np.array_equal(poly.cpu().numpy().astype(np.int64), np.asarray(want_poly).astype(np.int64))


@pytest.mark.parametrize("n", [1, 63, 64, 65, 511, 513, 2047, 2048, 2049, 4097, 100_003])
@pytest.mark.parametrize("overlap", [0.0, 0.004, 0.1, 0.5])
def test_pairs_match_oracle(ctx, n, overlap):
    """No overlap, one found on the way (few pixels in several polygons), and
    ones that the canvas shows beforehand."""
    polys = gen.rect_grid(12, 9, 0.0, 0.0, 1.0, 1.0)
    if overlap:
        polys = gen.concat_polys(polys, gen.star_polygon(60, overlap, (6.0, 4.5), L=9.0, seed=4))
    _check(ctx, *_points(n, 12, 9, n), polys)


@pytest.mark.parametrize("nx,ny", [(255, 257), (256, 256)])
def test_label_widths(ctx, nx, ny):
    """65,535 polygons fit 16 bits, 65,536 do not."""
    _check(ctx, *_points(20_001, nx, ny, nx), gen.rect_grid(nx, ny, 0.0, 0.0, 1.0, 1.0))
