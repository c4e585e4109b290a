"""A selection's estimate covers what it leaves on its worker: the canvas set
and the scratch that orders its ids (match bits and keys by table chunk)."""
import numpy as np
import pytest
import torch

from paper_2203_14362_amd.serve import Request, SpadeExecutor
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("area", [1e-5, 1e-3, 0.05, 0.4])
@pytest.mark.parametrize("n", [20_000, 4_000_000])
def test_selection_estimate(n, area):
    rng = np.random.default_rng(n)
    L = 1000.0
    x, y = (torch.from_numpy(rng.uniform(0, L, n)).cuda() for _ in range(2))
    ex = SpadeExecutor(x, y, n_workers=2)
    star = gen.star_polygon(24, area, (0.5 * L, 0.5 * L), L=L, seed=3)
    r = Request(0, "select", star)
    ex.run(1, [r])          # worker 0 made the table, whose scratch it keeps
    ex._measure_resident(1)
    assert 4 * r.result.numel() + ex._resident_w[1] <= ex.estimate(r)
    ex.close()
