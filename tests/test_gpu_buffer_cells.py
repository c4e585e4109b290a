"""The cells of the distance selections: fine cells that lie wholly within the
distance (many points) and the coarser ones of few points, lattice points at
exactly the distance (left open by the floating-point filter, which decides
first from 2^20 points on), segments much longer and much shorter than a cell, coordinates large beside the distance.
Ids are decided exactly, compared with the oracle's."""
import numpy as np
import pytest
import torch

from oracle import buffer as B
from workloads import gen

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _lines(rings):
    return gen.polys_from_rings([[np.asarray(r, dtype=np.float64)] for r in rings])


GEOMETRY = {
    "axis": [[[20, 40], [260, 40]], [[100, 10], [100, 290], [200, 290]]],
    "diagonal": [[[3, 5], [295, 291]]],
    "short": [[[20.0 + 13 * k, 30.0 + 11 * k], [20.5 + 13 * k, 30.0 + 11 * k], [20.5 + 13 * k, 30.5 + 11 * k]]
              for k in range(18)],
    "points": [[[10.0 + 17 * k, 280.0 - 15 * k]] for k in range(16)],
}


@pytest.mark.parametrize("n", [1, 65, 1023, 1025, 90_000, (1 << 20) - 1, (1 << 20) + 1])
@pytest.mark.parametrize("shape", sorted(GEOMETRY))
def test_lattice(ctx, n, shape):
    side = 300
    k = np.arange(n) * 7919 % (side * side)
    x, y = (k % side).astype(np.float64), (k // side).astype(np.float64)
    for r in (5.0, 13.0, 0.0):
        lines = _lines(GEOMETRY[shape])
        got = ctx.select_near_lines(_dev(x), _dev(y), lines, r).cpu().numpy().astype(np.int64)
        assert np.array_equal(got, B.select_near_lines(x, y, lines, r))


@pytest.mark.parametrize("shift", [0.0, 2.0 ** 30])
@pytest.mark.parametrize("r", [0.25, 4.0, 40.0])
def test_random(ctx, shift, r):
    rng = np.random.default_rng(int(r * 4))
    x, y = rng.uniform(-20, 320, 60_001) + shift, rng.uniform(-20, 320, 60_001) - shift
    rings = [np.asarray(s, dtype=np.float64) + [shift, -shift] for g in GEOMETRY.values() for s in g]
    lines = gen.polys_from_rings([[s] for s in rings])
    got = ctx.select_near_lines(_dev(x), _dev(y), lines, r).cpu().numpy().astype(np.int64)
    assert np.array_equal(got, B.select_near_lines(x, y, lines, r))


@pytest.mark.parametrize("r", [0.5, 6.0])
def test_polygon(ctx, r):
    poly = gen.star_polygon(40, 0.1, (150.0, 150.0), L=290.0, seed=7)
    k = np.arange(90_000)
    x, y = (k % 300).astype(np.float64), (k // 300).astype(np.float64)
    got = ctx.select_within(_dev(x), _dev(y), poly, r).cpu().numpy().astype(np.int64)
    assert np.array_equal(got, B.select_within_polygon(x, y, poly, r))
