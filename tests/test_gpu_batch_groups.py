"""Batch selection in groups: the scratch of many queries of one table chunk each
stays within what the limit on hit words allows, and a first group without any
(chunk, query) overlap leaves a valid timing."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_14362_amd import Context
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.fixture()
def own():
    c = Context(0)
    yield c
    c.close()


def _squares(nq, side, seed):
    rng = np.random.default_rng(seed)
    a = rng.uniform(0, 1 - side, (nq, 2))
    return gen.polys_from_rings([[np.array([[u, v], [u + side, v], [u + side, v + side], [u, v + side]])] for u, v in a])


def test_scratch_of_many_small_queries(own, monkeypatch):
    nq, limit = 3000, 1 << 18
    rng = np.random.default_rng(4)
    x, y = rng.uniform(0, 1, 200_000), rng.uniform(0, 1, 200_000)
    polys = _squares(nq, 0.004, 5)
    t = own.table(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    b = own.batch(polys, np.arange(nq + 1))
    monkeypatch.setenv("SPADE_HIT_MASK_LIMIT", str(limit))
    before = own.mem_info()["ctx"]
    ids, off = own.batch_select(b, t)
    # keys of 16 KB per 512 bytes of hit words, a quarter more than asked for,
    # and small lists
    assert own.mem_info()["ctx"] - before < 40 * limit + (4 << 20)
    got = ids.cpu().numpy().astype(np.int64)
    for q in range(0, nq, 37):
        assert np.array_equal(got[off[q]:off[q + 1]], oracle.select(x, y, polys, q).astype(np.int64))
    monkeypatch.delenv("SPADE_HIT_MASK_LIMIT")
    ids2, off2 = own.batch_select(b, t)
    assert np.array_equal(off, off2) and torch.equal(ids, ids2)


@pytest.mark.parametrize("limit", [None, "0"])
def test_timing_without_overlaps(own, monkeypatch, limit):
    if limit is not None:
        monkeypatch.setenv("SPADE_HIT_MASK_LIMIT", limit)
    p = torch.rand(5000, device="cuda", dtype=torch.float64)
    t = own.table(p, p.flip(0).contiguous())
    far = _squares(3, 0.1, 6)
    far["vx"] = far["vx"] + 7.0
    b = own.batch(far, np.arange(4))
    own.set_timing(True)
    ids, off = own.batch_select(b, t)
    assert ids.numel() == 0 and not off.any()
    assert 0.0 <= own.last_timing()[1] < 1000.0
