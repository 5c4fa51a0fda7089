"""The bound of the k-th distance from the sample: batches that fill few and many of the sample pass's workgroups (waves
that share a stretch of the sample, sub-tiles past the last query), and every size class of the bound kernel, checked
against the exact whole-database selection of the same library, which the oracle's tests pin."""
import numpy as np
import pytest

from test_gpu_parity import FLAT, FOREST, Problem, say, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def problem():
    return Problem(d=16, M=8, K=256, N=40000, Q=1100, ntrain=4000, seed=31)


@pytest.fixture(scope="module")
def problem16():
    return Problem(d=32, M=16, K=256, N=30000, Q=130, ntrain=4000, seed=32)


def check(p, Q, k, mode, T, **opts):
    qd = torch.from_numpy(p.q[:Q]).cuda()
    c = p.ctx(T=T, sample_min=1 << 14, cand_cap=8192, **opts)
    ids, dist = c.search(qd, k, mode)
    torch.cuda.synchronize()
    assert c.last_fallback_count() == 0
    c.set_option("force_fallback", 1)
    wi, wd = c.search(qd, k, mode)
    torch.cuda.synchronize()
    assert c.last_fallback_count() == Q
    assert torch.equal(dist, wd) and torch.equal(ids, wi)


# 1 query, a sub-tile, a tile and their neighbours, a chip's worth of sub-tiles; group counts 1024, 2048 and 4096 (k)
@pytest.mark.parametrize("Q", [1, 16, 17, 64, 65, 1100])
@pytest.mark.parametrize("k", [1, 409, 410, 820, 1000])
def test_bound_sizes(problem, Q, k):
    say("bound Q", Q, "k", k)
    check(problem, Q, k, FOREST, 2)


# the other writers of the group minima: flat scan, 16-byte codes, the table-based traversals (256 groups)
@pytest.mark.parametrize("mode,T,trav", [(FLAT, 1, 2), (FLAT, 1, 0), (FOREST, 2, 0), (FOREST, 2, 1)])
@pytest.mark.parametrize("k", [3, 200])
def test_bound_writers(problem, mode, T, trav, k):
    say("bound mode", mode, "traversal", trav, "k", k)
    check(problem, 150, k, mode, T, traversal=trav)


@pytest.mark.parametrize("Q", [1, 8, 9, 130])
def test_bound_sixteen_chunks(problem16, Q):
    say("bound M = 16, Q", Q)
    check(problem16, Q, 20, FOREST, 4)


# scalar products: the tables shifted by their maxima, whose sum is subtracted again
@pytest.mark.parametrize("Q", [1, 65])
@pytest.mark.parametrize("K", [3, 100, 256])
def test_products_shift(K, Q):
    say("products K", K, "Q", Q)
    p = Problem(d=24, M=4, K=K, N=9000, Q=Q, ntrain=1000, seed=33)
    check(p, Q, 30, FOREST, 1, metric=1)
