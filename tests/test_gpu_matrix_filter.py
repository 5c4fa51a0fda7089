"""The filter pass on the matrix cores (k_mm16): chunks of 1 to 8 dimensions, batches around its blocks of 128 queries, indexes
that end inside a step of 32 encodings, chunk orders, and blocks it leaves to the table kernel because its error bound is
not small against the distances.  It only selects: ids and float32 distances are those of the exact whole-database
selection, bit for bit, and no query may need that selection."""
import numpy as np
import pytest

from workload import GaussianMixture
from test_gpu_parity import FOREST, TREE, Problem, etf, say, torch

pytestmark = pytest.mark.gpu


def check(c, q, k, mode, fallback=0, taken=None):
    """taken: blocks of 128 queries that k_mm16 must have filtered (all of them unless given)."""
    qd = torch.from_numpy(q).cuda()
    ids, dist = c.search(qd, k, mode)
    torch.cuda.synchronize()
    assert c.last_fallback_count() == fallback
    assert c.last_matrix_blocks() == ((len(q) + 127) // 128 if taken is None else taken)
    c.set_option("lds_filter", 0)
    ids0, dist0 = c.search(qd, k, mode)
    torch.cuda.synchronize()
    assert c.last_matrix_blocks() == 0
    c.set_option("force_fallback", 1)
    wi, wd = c.search(qd, k, mode)
    torch.cuda.synchronize()
    assert c.last_fallback_count() == len(q)
    c.set_option("force_fallback", 0)
    c.set_option("lds_filter", 2)
    assert torch.equal(dist, dist0) and torch.equal(ids, ids0)
    assert torch.equal(dist, wd) and torch.equal(ids, wi)


def filled(M, Q):
    """Blocks of a batch of ordinary queries that k_mm16 takes: all, where the batch fills them beside sub-tiles of 32 (M = 8) or
    16 queries to at most half as much again."""
    sub, blocks = (32 if M == 8 else 16), (Q + 127) // 128
    return blocks if 2 * 128 * blocks <= 3 * sub * ((Q + sub - 1) // sub) else 0


@pytest.mark.parametrize("M,ds,T,N,k", [(16, 8, 4, 30001, 20), (16, 5, 1, 29999, 20), (16, 1, 2, 20031, 900), (8, 8, 2, 40000, 20),
                                        (8, 3, 1, 33333, 200)])
def test_shapes_and_block_edges(M, ds, T, N, k):
    say("matrix filter M", M, "ds", ds, "T", T, "N", N)
    p = Problem(d=M * ds, M=M, K=256, N=N, Q=400, ntrain=3000, seed=M + ds)
    c = p.ctx(matrix_filter=0, T=T, sample_min=1 << 13, cand_cap=8192)
    for Q in (86, 96, 127, 128, 129, 192, 257, 400):  # the smallest batches that take it, and the edges of its blocks
        check(c, p.q[:Q], k, TREE if T == 1 else FOREST, taken=filled(M, Q))


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


def with_a_tight_cluster(M, ds, N, Q, seed):
    """A problem whose first two codewords of every chunk nearly coincide and of whose database a sixth is made of them:
    a query at such a reconstruction has distances far below the matrix filter's error bound."""
    p = Problem(d=M * ds, M=M, K=256, N=N, Q=Q, ntrain=3000, seed=seed)
    rng = np.random.default_rng(seed)
    p.cb[:, 1] = p.cb[:, 0] * np.float32(1 + 1e-4)
    p.codes[:N // 6] = rng.integers(0, 2, (N // 6, M))
    return p, p.cb[:, 0].reshape(-1)


@pytest.mark.parametrize("M,T", [(16, 4), (8, 2)])
def test_blocks_left_to_the_table_filter(M, T):
    say("matrix filter: blocks left to the table kernel, beside blocks that are not, M", M)
    p, tight = with_a_tight_cluster(M, 8, 30000, 700, 51)
    c = p.ctx(matrix_filter=0, T=T, sample_min=1 << 14, cand_cap=8192)
    for at in ([], [0], [699], [130, 131, 200], [5, 300, 650], [0, 130, 260], [383, 384, 520], [0, 130, 260, 390], range(0, 700, 100), range(0, 700, 64)):
        q = p.q.copy()
        q[list(at)] = tight
        own = 6 - len({i // 128 for i in at})
        check(c, q, 10, FOREST, taken=own if 2 * own >= 6 else 0)  # fewer than half are not worth a kernel of their own
    q = p.q.copy()
    q[[130, 650]] = tight
    for blocks in (1, 5, 40):           # workgroups per unit by the option in place of the rule
        c.set_option("lds_blocks", blocks)
        check(c, q, 10, FOREST, taken=4)


def test_replays_divide_the_batch_anew():
    say("matrix filter: a captured search on other queries, other blocks left to the table kernel every time")
    p, tight = with_a_tight_cluster(16, 8, 30000, 700, 53)
    c = p.ctx(matrix_filter=0, T=4, sample_min=1 << 14, cand_cap=8192)
    k, qd = 10, torch.from_numpy(p.q).cuda()
    ws = c.alloc_workspace(700, k, FOREST)
    ids = torch.zeros((700, k), dtype=torch.int32, device="cuda")
    dist = torch.zeros((700, k), dtype=torch.float32, device="cuda")
    c.search(qd, k, FOREST, ids, dist, ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        c.set_stream(torch.cuda.current_stream().cuda_stream)
        c.search(qd, k, FOREST, ids, dist, ws)
    c.set_stream(torch.cuda.current_stream().cuda_stream)
    for at, taken in (([5, 300], 4), ([], 6), (range(0, 700, 64), 0), ([699], 5), ([0, 130, 260, 390], 0), ([], 6)):
        q = torch.from_numpy(p.q).cuda()
        q[list(at)] = torch.from_numpy(tight).cuda()
        qd.copy_(q)
        g.replay()
        torch.cuda.synchronize()
        assert c.last_matrix_blocks() == taken and c.last_fallback_count() == 0
        c.set_option("matrix_filter", -1)
        want_i, want_d = c.search(q, k, FOREST)
        torch.cuda.synchronize()
        c.set_option("matrix_filter", 0)
        assert torch.equal(ids, want_i) and torch.equal(dist, want_d)
        c.search(q, k, FOREST, want_i, want_d, ws)          # eager work on the same workspace, counts in place again
        torch.cuda.synchronize()
        assert c.last_matrix_blocks() == taken


def test_batches_of_a_small_workspace():
    """The blocks, their words and their counts belong to a batch of tiles: several batches, the last one of a single tile."""
    say("matrix filter: one search in several batches")
    p, tight = with_a_tight_cluster(8, 8, 30000, 1100, 54)
    q = p.q.copy()
    q[[130, 400, 900]] = tight
    c = p.ctx(matrix_filter=0, T=2, sample_min=1 << 14, cand_cap=8192)
    qd = torch.from_numpy(q).cuda()
    want_i, want_d = c.search(qd, 10, FOREST)
    torch.cuda.synchronize()
    for tiles in (3, 4, 7):
        c.set_option("ws_cap_bytes", int(c.alloc_workspace(64, 10, FOREST).numel() * (tiles + 0.5)))
        ids, dist = c.search(qd, 10, FOREST)
        torch.cuda.synchronize()
        assert c.last_fallback_count() == 0
        say("  batches of", tiles, "tiles:", c.last_matrix_blocks(), "blocks on the matrix cores")
        assert torch.equal(ids, want_i) and torch.equal(dist, want_d)
    ids.zero_()
    c.search_static(qd, 10, FOREST, ids, dist)
    torch.cuda.synchronize()
    assert torch.equal(ids, want_i) and torch.equal(dist, want_d)


def test_outliers():
    say("matrix filter: one query far out (the scale of its block), one at the origin")
    p = Problem(d=128, M=16, K=256, N=30000, Q=384, ntrain=3000, seed=51)
    q = p.q.copy()
    q[300] *= 1000.0
    q[301] = 0.0
    check(p.ctx(matrix_filter=0, T=4, sample_min=1 << 14, cand_cap=8192), q, 10, FOREST)


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


@pytest.mark.parametrize("M,T", [(16, 4), (8, 2)])
def test_candidates_fit_where_those_of_the_table_filter_do(M, T):
    """k_mm16 lets everything up to tau + E through.  With lists from far too short to the default length, no more queries may
    need the exact selection than with the table filter; with room for them all, the blocks are taken."""
    say("matrix filter: candidate lists, M", M)
    gm = GaussianMixture(8 * M, 64, 1.1, (0.2, 1.0), (-4.0, 4.0), seed=60)
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    c.pq_train(gm.sample(4000, 1), M, 256, 3, 1)
    N, Q, k = 300_000, 512, 100
    c.index_build_device(c.pq_encode_device(torch.from_numpy(gm.sample(N, 2)).cuda()), T=T)
    q = torch.from_numpy(gm.sample(Q, 3)).cuda()
    over = {}
    for cap in (256, 384, 512, 640, 768, 1024, 1280, 1536, 2048, 0):
        c.set_option("cand_cap", cap)
        for pairs in (-1, 0):
            c.set_option("matrix_filter", pairs)
            c.search(q, k, FOREST)
            torch.cuda.synchronize()
            over[cap, pairs] = c.last_fallback_count()
        say("  cap", cap, "exact selections: table", over[cap, -1], "matrix", over[cap, 0])
    assert all(over[cap, 0] <= over[cap, -1] for cap, _ in over)
    assert over[0, 0] == 0 and c.last_matrix_blocks() == Q // 128
    c.set_option("cand_cap", 256)
    c.search(q, k, FOREST)
    torch.cuda.synchronize()
    assert c.last_matrix_blocks() == 0
