"""The filter pass on the matrix cores (k_mm16): chunks of 1 to 8 dimensions, batches around its blocks of 128 queries, indexes
that end inside a step of 32 encodings, chunk orders, and blocks it leaves to the table kernel because its error bound is
not small against the distances.  It only selects: ids and float32 distances are those of the exact whole-database
selection, bit for bit, and no query may need that selection."""
import numpy as np
import pytest

from test_gpu_parity import FOREST, TREE, Problem, etf, say, torch

pytestmark = pytest.mark.gpu


def check(c, q, k, mode, fallback=0):
    qd = torch.from_numpy(q).cuda()
    ids, dist = c.search(qd, k, mode)
    torch.cuda.synchronize()
    assert c.last_fallback_count() == fallback
    c.set_option("lds_filter", 0)
    ids0, dist0 = c.search(qd, k, mode)
    c.set_option("force_fallback", 1)
    wi, wd = c.search(qd, k, mode)
    torch.cuda.synchronize()
    assert c.last_fallback_count() == len(q)
    c.set_option("force_fallback", 0)
    c.set_option("lds_filter", 2)
    assert torch.equal(dist, dist0) and torch.equal(ids, ids0)
    assert torch.equal(dist, wd) and torch.equal(ids, wi)


@pytest.mark.parametrize("M,ds,T,N", [(16, 8, 4, 30001), (16, 5, 1, 29999), (16, 1, 2, 20031), (8, 8, 2, 40000), (8, 3, 1, 33333)])
def test_shapes_and_block_edges(M, ds, T, N):
    say("matrix filter M", M, "ds", ds, "T", T, "N", N)
    p = Problem(d=M * ds, M=M, K=256, N=N, Q=400, ntrain=3000, seed=M + ds)
    c = p.ctx(matrix_filter=0, T=T, sample_min=1 << 13, cand_cap=8192)
    for Q in (86, 96, 127, 128, 129, 400):  # the smallest batches that take it, and the edges of its blocks
        check(c, p.q[:Q], 20, TREE if T == 1 else FOREST)


@pytest.mark.parametrize("k", [1, 100, 900])
def test_k_and_chunk_order(k):
    say("matrix filter k", k)
    p = Problem(d=64, M=8, K=200, N=35000, Q=256, ntrain=3000, seed=50)
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    c.set_option("sample_min", 1 << 14)
    c.set_option("matrix_filter", 0)
    c.set_option("cand_cap", 16384)
    c.pq_set_codebooks(p.cb)
    c.index_set_chunk_order([3, 1, 7, 5, 0, 2, 6, 4])
    c.index_build(p.codes, T=2)
    c.index_upload()
    check(c, p.q, k, FOREST)


def test_clusters_far_from_the_mean_and_outliers():
    say("matrix filter: blocks left to the table kernel, beside blocks that are not")
    p = Problem(d=128, M=16, K=256, N=30000, Q=384, ntrain=3000, seed=51)
    q = p.q.copy()
    q[128:256] = p.xb[:128]                 # distances near zero: no bound is small against them
    q[300] *= 1000.0                        # one query far out: the block's scale, and a bound of its own
    q[301] = 0.0
    c = p.ctx(matrix_filter=0, T=4, sample_min=1 << 14, cand_cap=8192)
    check(c, q, 10, FOREST)


def test_queries_that_are_not_finite():
    say("matrix filter: NaN and infinities beside ordinary queries")
    p = Problem(d=64, M=8, K=256, N=30000, Q=256, ntrain=3000, seed=52)
    c = p.ctx(matrix_filter=0, T=2, sample_min=1 << 13, cand_cap=8192)
    want = c.search(torch.from_numpy(p.q).cuda(), 10, FOREST)
    q = p.q.copy()
    q[5, 3], q[130, 0], q[131, 63] = np.nan, np.inf, -np.inf
    got = c.search(torch.from_numpy(q).cuda(), 10, FOREST)
    torch.cuda.synchronize()
    keep = torch.from_numpy(np.isfinite(q).all(1)).cuda()
    assert torch.equal(got[0][keep], want[0][keep]) and torch.equal(got[1][keep], want[1][keep])
