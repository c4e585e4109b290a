"""Join-counts of more polygons than the probe's LDS histogram holds (8,192),
which are counted through 16-bit labels up to 65,535 polygons: sizes around a
counting round (8,192 labels), points in several polygons, a counter driven
past 16 bits and the largest polygon counts.  Counts are whole numbers decided
exactly, compared with the oracle's or a closed form."""
import numpy as np
import pytest
import torch

import oracle
from workloads import gen

pytestmark = pytest.mark.gpu


def _grid_cells(nx, ny):
    return gen.rect_grid(nx, ny, 0.0, 0.0, 1.0, 1.0)


@pytest.mark.parametrize("n", [1, 7, 8191, 8193, 65537, 300_001])
@pytest.mark.parametrize("overlap", [False, True])
def test_counts_match_oracle(ctx, n, overlap):
    rng = np.random.default_rng(n)
    cells = _grid_cells(96, 90)     # 8,640 cells
    if overlap:                     # a tenth of them lies under a star as well
        star = gen.star_polygon(60, 0.1, (48.0, 45.0), L=90.0, seed=4)
        cells = gen.concat_polys(cells, star)
    x, y = rng.uniform(-2, 98, n), rng.uniform(-2, 92, n)
    x[::97], y[::89] = np.round(x[::97]), np.round(y[::89])   # on cell sides
    if n > 10:
        x[3], y[5] = np.nan, np.inf
    got = ctx.join_count(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), cells)
    assert np.array_equal(got.cpu().numpy().astype(np.uint64), oracle.join_count(x, y, cells))


def test_counter_past_16_bits(ctx):
    """Nearly all points in one cell: every workgroup's counter passes 2^15
    more than once."""
    cells = _grid_cells(100, 90)
    n = 256 * 8192 * 12 + 5
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = 7.0 + 0.999 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    y = 5.0 + 0.999 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    y[::1000] += 1.0
    got = ctx.join_count(x, y, cells).cpu().numpy()
    want = np.zeros(9000, dtype=np.int64)
    moved = (n + 999) // 1000
    k = [int(np.argmax(oracle.join_count(np.array([7.5]), np.array([v]), cells))) for v in (5.5, 6.5)]
    want[k[0]], want[k[1]] = n - moved, moved
    assert np.array_equal(got, want)


@pytest.mark.parametrize("nx,ny", [(255, 257), (256, 256)])
def test_most_labels(ctx, nx, ny):
    """65,535 polygons have labels, 65,536 do not."""
    cells = _grid_cells(nx, ny)
    rng = np.random.default_rng(nx)
    x, y = rng.uniform(0, nx, 100_000), rng.uniform(0, ny, 100_000)
    got = ctx.join_count(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), cells)
    assert np.array_equal(got.cpu().numpy().astype(np.uint64), oracle.join_count(x, y, cells))
