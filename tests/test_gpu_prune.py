"""Searches on queries put in order and on the parts of the index that a group of them needs (k_order_*, k_prune, k_units and
the two walks of k_lds16 over lists).  They only leave out what cannot be among the k nearest: ids and float32 distances are those
of the float32 filter over everything and of the exact whole-database selection, bit for bit, and no query may need the latter.
Sizes lie around the blocks of 64 encodings, the sub-tiles of 32 and 16 queries and the blocks of 128."""
import numpy as np
import pytest

from test_host_order_plan import clusters, context, near
from test_gpu_parity import FOREST, TREE, Problem, etf, say, torch

pytestmark = pytest.mark.gpu


def check(c, q, k, mode, fallback=0):
    qd = torch.from_numpy(q).cuda()
    c.set_option("prune_filter", -1)
    plain = c.workspace_bytes(len(q), k, mode)
    c.set_option("prune_filter", 0)
    assert c.workspace_bytes(len(q), k, mode) != plain  # it has lists
    ids, dist = c.search(qd, k, mode)
    torch.cuda.synchronize()
    assert c.last_fallback_count() == fallback
    assert c.last_kept_encodings() > 0 or c.last_matrix_blocks() > 0
    c.set_option("lds_filter", 0)
    ids0, dist0 = c.search(qd, k, mode)
    assert c.last_kept_encodings() == 0
    c.set_option("force_fallback", 1)
    wi, wd = c.search(qd, k, mode)
    torch.cuda.synchronize()
    c.set_option("force_fallback", 0)
    c.set_option("lds_filter", 2)
    assert torch.equal(dist, dist0) and torch.equal(ids, ids0)
    assert torch.equal(dist, wd) and torch.equal(ids, wi)


@pytest.mark.parametrize("M,ds,T,N,Q,k", [(8, 4, 2, 20000, 1, 10), (8, 4, 1, 20031, 33, 1), (8, 3, 2, 20032, 129, 100), (8, 16, 2, 30001, 400, 300),
                                          (16, 2, 4, 20063, 17, 10), (16, 4, 1, 20064, 130, 50), (16, 1, 2, 30000, 257, 900)])
def test_shapes_and_block_edges(M, ds, T, N, Q, k):
    p = Problem(d=M * ds, M=M, K=256, N=N, Q=Q, ntrain=3000, seed=M + ds)
    check(p.ctx(T=T, sample_min=1 << 13, cand_cap=16384 if k > 500 else 8192, matrix_filter=-1), p.q, k, TREE if T == 1 else FOREST)


@pytest.mark.parametrize("M,K", [(8, 200), (16, 137)])
def test_fewer_codewords_and_a_chunk_order(M, K):
    p = Problem(d=4 * M, M=M, K=K, N=25000, Q=150, ntrain=3000, seed=7)
    c = p.ctx(T=1, sample_min=1 << 13, cand_cap=8192, matrix_filter=-1)
    c.index_set_chunk_order(list(range(M))[::-1])
    c.index_build(p.codes, T=2)
    c.index_upload()
    check(c, p.q, 20, FOREST)


def test_clusters_of_few_encodings():
    """Vectors of tight clusters share encodings: fewer than k of them hold a query's k neighbours."""
    p = Problem(d=32, M=8, K=256, N=24000, Q=300, ntrain=3000, seed=3)
    rng = np.random.default_rng(1)
    p.codes[:12000] = p.codes[rng.integers(12000, 12040, 12000)]  # 300 vectors an encoding
    near = rng.integers(12000, 12040, 100)
    p.q[:100] = p.xb[near] + rng.normal(0, 1e-3, (100, 32)).astype(np.float32)
    check(p.ctx(T=2, sample_min=1 << 13, cand_cap=8192), p.q, 200, FOREST)


def clustered(N, M, **opts):
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    for name, v in opts.items():
        c.set_option(name, v)
    cb, codes = clusters(N, M)
    c.pq_set_codebooks(cb)
    c.index_build_device(torch.from_numpy(codes).cuda(), T=2)
    assert c.index_stats()["n_distinct"] == N
    return c, cb, codes


@pytest.mark.parametrize("M", [8, 16])
@pytest.mark.parametrize("N", [64 * 313, 64 * 313 + 1, 64 * 313 + 63])
@pytest.mark.parametrize("Q", [256, 1100])   # at M = 8: two workgroups for the closer bound of a sub-tile, one
def test_edges_of_the_distinct_encodings(M, N, Q):
    c, cb, codes = clustered(N, M, sample_min=1 << 13, cand_cap=8192, matrix_filter=-1)
    check(c, near(cb, codes, Q), 10, FOREST)


@pytest.mark.parametrize("M,shift,over", [(8, 1, 1), (8, 1, 64), (8, 1, 128 * 7), (8, 2, 65), (8, 2, 193), (16, 1, 127), (16, 2, 256 * 3 + 64)])
def test_blocks_of_several_runs_of_64(M, shift, over):
    """Above 2^16 x 64 encodings a block of the lists is 2 or 4 runs of 64, the last of which may lie past the end of the index."""
    N = (1 << (21 + shift)) + over
    c, cb, codes = clustered(N, M, matrix_filter=-1, prune_filter=0)
    last = near(cb, codes[-64:], 8, seed=2)   # (the highest numbers; and vectors of the last encodings in the tree's order)
    end = codes[np.lexsort(codes[:, ::-1].T)[-200:]]
    q = torch.from_numpy(np.concatenate([near(cb, codes, 130), last, near(cb, end, 64, seed=3)])).cuda()
    got = c.search(q, 20, FOREST)
    assert c.last_fallback_count() == 0
    group = 32 if M == 8 else 16
    kept, whole = c.last_kept_encodings(), -(-len(q) // group) * N
    say("kept %.3f" % (kept / whole))
    assert 0 < kept < 0.5 * whole and kept % (64 << shift) == 0
    c.set_option("prune_filter", -1)
    want = c.search(q, 20, FOREST)
    assert c.last_kept_encodings() == 0
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("M", [8, 16])
def test_a_bound_that_the_nearest_blocks_do_not_better(M):
    """The first three chunks tell nothing (their codewords are as good as one), the lists have room for what the whole sample's
    bound lets through (1.3 k N / S = 2400) and no more: no query may overrun its list."""
    rng = np.random.default_rng(3)
    cb = rng.normal(0, 1, (M, 256, 4)).astype(np.float32)
    cb[:3] *= 1e-3
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    for name, v in (("cand_cap", 4096), ("matrix_filter", -1)):
        c.set_option(name, v)
    c.pq_set_codebooks(cb)
    c.index_build(rng.integers(0, 256, (200000, M)).astype(np.uint8), T=2)
    c.index_upload()
    check(c, rng.normal(0, 1, (200, 4 * M)).astype(np.float32), 500, FOREST)


@pytest.mark.parametrize("M,far,k,mm", [(8, 1, 10, -1), (8, 300, 100, -1), (16, 1, 20, -1), (16, 37, 1, 0), (16, 300, 300, -1)])
def test_queries_whose_lists_overrun(M, far, k, mm):
    """All distances from a query far away lie within the rounding of the 16-bit tables: every encoding is at or below its bound.  Its list
    is made anew with the k-th distance of what the first one held; nothing is left to the exact selection, also in repeated calls.
    (What a list of C = 16384 of the N = 30000 encodings holds is a matter of the schedule; at least 2 C - N = 2768 >= k of the nearest C are
    among them, so that at most C lie at or below the k-th.)"""
    N, Q = 30000, 300
    cb, codes = clusters(N, M)
    q = near(cb, codes, Q)
    q[np.random.default_rng(1).permutation(Q)[:far]] += 20000.0
    c = context(N, M, device=0, matrix_filter=mm, sample_min=1 << 13, cand_cap=16384)
    c.set_stream(torch.cuda.current_stream().cuda_stream)
    c.index_upload()
    check(c, q, k, FOREST)
    qd = torch.from_numpy(q).cuda()
    c.set_option("prune_filter", -1)
    want = c.search(qd, k, FOREST)
    assert c.last_fallback_count() >= far
    c.set_option("prune_filter", 0)
    c.set_option("ws_cap_bytes", int(c.workspace_bytes(64, k, FOREST) * 2.5))   # batches of two tiles
    got = c.search(qd, k, FOREST)
    assert c.last_fallback_count() == 0
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_lists_that_overrun_twice():
    """1000 neighbours in a list of 2048 out of 30 000: some 15 000 encodings are at or below the second bound, unless the first list happened to hold
    half of the nearest ones, which it does not for 64 queries in different directions."""
    N, M = 30000, 8
    cb, codes = clusters(N, M)
    rng = np.random.default_rng(5)
    q = near(cb, codes, 70)
    q[:64] += (20000.0 * rng.choice([-1, 1], (64, q.shape[1]))).astype(np.float32)
    c = context(N, M, device=0, matrix_filter=-1, sample_min=1 << 13, cand_cap=2048, prune_filter=0)
    c.set_stream(torch.cuda.current_stream().cuda_stream)
    c.index_upload()
    qd = torch.from_numpy(q).cuda()
    got = c.search(qd, 1000, FOREST)
    say("exact selections", c.last_fallback_count())
    assert c.last_fallback_count() > 0 and c.last_kept_encodings() > 0
    c.set_option("force_fallback", 1)
    want = c.search(qd, 1000, FOREST)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_beside_the_matrix_filter():
    p = Problem(d=128, M=16, K=256, N=30000, Q=400, ntrain=3000, seed=5)
    check(p.ctx(T=4, sample_min=1 << 14, cand_cap=8192, matrix_filter=0), p.q, 20, FOREST)


def test_the_matrix_filter_and_the_lists_share_a_batch():
    """Two blocks of 128 queries beside vectors of the index, which keep little, and two of queries far from everything, which keep it all.  The
    latter lie at a group of codewords of the first chunk that no vector has, so that they come last."""
    M, N = 16, 30000
    cb, codes = clusters(N, M)
    codes[:, 0] %= 248
    rng = np.random.default_rng(6)
    far = rng.normal(0, 3, (256, M, 4)).astype(np.float32)
    far[:, 0] = cb[0, 248:].mean(axis=0)
    q = np.concatenate([near(cb, codes, 256), far.reshape(256, -1)])[rng.permutation(512)]
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    for name, v in (("sample_min", 1 << 13), ("cand_cap", 8192), ("matrix_filter", 0), ("prune_filter", 0)):
        c.set_option(name, v)
    c.pq_set_codebooks(cb)
    c.index_build(codes, T=2)
    c.index_upload()
    c.search(torch.from_numpy(q).cuda(), 20, FOREST)
    say("blocks on the matrix cores", c.last_matrix_blocks(), "kept", c.last_kept_encodings())
    assert 0 < c.last_matrix_blocks() < 4 and c.last_kept_encodings() > 0
    check(c, q, 20, FOREST)


def test_workspaces_of_larger_calls():
    """One workspace for the largest call serves the smaller ones: on queries in order where it holds that plan, else as they come."""
    c = context(300000, device=0, prune_filter=1)
    c.set_stream(torch.cuda.current_stream().cuda_stream)
    c.index_upload()
    q = torch.randn((1100, 32), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    for Q, k, n, m, ordered in ((1100, 101, 1100, 99, False), (1100, 300, 1000, 50, False), (1100, 300, 1000, 10, True), (1100, 100, 1001, 100, True), (1100, 100, 999, 100, False)):
        ws = c.alloc_workspace(Q, k, FOREST)
        ids, dist = c.search(q[:n], m, FOREST, ws=ws)
        assert (c.last_kept_encodings() > 0) == ordered
        own = c.search(q[:n], m, FOREST)
        assert (c.last_kept_encodings() > 0) == (n >= 1000)
        assert torch.equal(ids, own[0]) and torch.equal(dist, own[1])
    ws = torch.empty(c.workspace_bytes(1100, 101, FOREST) - 256, dtype=torch.uint8, device="cuda")
    with pytest.raises(etf.EtfError):
        c.search(q, 101, FOREST, ws=ws[(-ws.data_ptr()) % 256:])


def test_batches_of_a_small_workspace():
    p = Problem(d=32, M=8, K=256, N=20000, Q=300, ntrain=3000, seed=9)
    c = p.ctx(T=2, sample_min=1 << 13, cand_cap=4096, prune_filter=0)
    c.set_option("ws_cap_bytes", int(c.workspace_bytes(64, 10, FOREST) * 2.5))
    check(c, p.q, 10, FOREST)


def test_more_sub_tiles_than_a_grid_has_rows():
    """A batch of a million queries, 65 537 groups of 16: more than the 65 535 workgroups that a launch may have along y."""
    N, M, Q = 20000, 16, 65536 * 16 + 5
    rng = np.random.default_rng(11)
    cb, codes = clusters(N, M)
    cb = np.ascontiguousarray(cb[:, :, :1])     # one dimension a chunk: small queries
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    for name, v in (("cand_cap", 2048), ("sample_min", 1 << 13), ("matrix_filter", -1), ("prune_filter", 0), ("ws_cap_bytes", 1 << 36)):
        c.set_option(name, v)
    c.pq_set_codebooks(cb)
    c.index_build(codes, T=2)
    c.index_upload()
    assert c.workspace_bytes(Q, 5, FOREST) < 1 << 36   # (one batch)
    q = torch.from_numpy(near(cb, codes, 4096)).cuda()[torch.from_numpy(rng.integers(0, 4096, Q)).cuda()]
    q += torch.randn(q.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(2)) * 0.01
    got = c.search(q, 5, FOREST)
    kept = c.last_kept_encodings()
    say("kept %.3f" % (kept / (65537 * N)), "exact selections", c.last_fallback_count())
    assert kept > 0
    c.set_option("prune_filter", -1)
    c.set_option("ws_cap_bytes", 1 << 33)
    want = c.search(q, 5, FOREST)
    assert c.last_kept_encodings() == 0
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("M,group", [(8, 32), (16, 16)])
def test_the_count_of_what_was_looked_at(M, group):
    """Codes without structure and a large k: every group of queries keeps every block of 64, in one batch and in several."""
    rng = np.random.default_rng(4)
    N, Q = 20001, 333
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    for name, v in (("cand_cap", 16384), ("matrix_filter", -1), ("sample_min", 1 << 13), ("prune_filter", 0)):
        c.set_option(name, v)
    c.pq_set_codebooks(rng.normal(0, 1, (M, 256, 4)).astype(np.float32))
    c.index_build(rng.integers(0, 256, (N, M)).astype(np.uint8), T=2)
    c.index_upload()
    q = torch.from_numpy(rng.normal(0, 1, (Q, 4 * M)).astype(np.float32)).cuda()
    for cap in (8 << 30, int(c.workspace_bytes(64, 900, FOREST) * 2.5)):
        c.set_option("ws_cap_bytes", cap)
        c.search(q, 900, FOREST)
        assert c.last_kept_encodings() == -(-Q // group) * -(-N // 64) * 64


def test_queries_that_are_not_finite():
    p = Problem(d=32, M=8, K=256, N=20000, Q=200, ntrain=3000, seed=13)
    c = p.ctx(T=2, sample_min=1 << 13, cand_cap=8192)
    want = c.search(torch.from_numpy(p.q).cuda(), 10, FOREST)
    bad = p.q.copy()
    bad[5], bad[40, 3], bad[190] = np.nan, np.inf, 3e38
    c.set_option("prune_filter", 0)
    got = c.search(torch.from_numpy(bad).cuda(), 10, FOREST)
    torch.cuda.synchronize()
    keep = [i for i in range(200) if i not in (5, 40, 190)]
    assert torch.equal(got[0][keep], want[0][keep]) and torch.equal(got[1][keep], want[1][keep])


@pytest.mark.parametrize("M,mm", [(8, -1), (16, -1), (16, 0)])
def test_a_query_that_is_not_finite_costs_its_neighbours_nothing(M, mm):
    """Such a query (a NaN or an infinity in one chunk, squares that are infinite) takes the exact selection, and its sub-tile keeps what
    the others need."""
    N, Q = 30000, 400
    cb, codes = clusters(N, M)
    q = near(cb, codes, Q)
    c = context(N, M, device=0, prune_filter=0, matrix_filter=mm, sample_min=1 << 13, cand_cap=8192)
    c.set_stream(torch.cuda.current_stream().cuda_stream)
    c.index_upload()
    bad = q.copy()
    bad[7, 5], bad[99], bad[150, :4], bad[251, 8], bad[333] = np.nan, np.nan, np.inf, -np.inf, 3e38
    wrong = [7, 99, 150, 251, 333]
    fine = [i for i in range(Q) if i not in wrong]
    want = c.search(torch.from_numpy(q).cuda(), 10, FOREST)
    clean = c.last_kept_encodings()
    got = c.search(torch.from_numpy(bad).cuda(), 10, FOREST)
    kept = c.last_kept_encodings()
    assert c.last_fallback_count() == len(wrong)
    assert torch.equal(got[0][fine], want[0][fine]) and torch.equal(got[1][fine], want[1][fine])
    c.set_option("prune_filter", -1)
    plain = c.search(torch.from_numpy(bad).cuda(), 10, FOREST)
    assert torch.equal(got[0], plain[0]) and torch.equal(got[1].nan_to_num(), plain[1].nan_to_num())
    whole = 30016 * ((Q * M // 4 + 63) // 64)   # encodings that all sub-tiles look at when nothing is left out
    say("kept", clean, kept, "of", whole)
    assert 0 < clean < 0.3 * whole
    assert kept < clean + 0.05 * whole          # (five sub-tiles that keep everything: a fifth or a tenth; the order moves a little)


def test_replays_of_a_graph():
    p = Problem(d=32, M=8, K=256, N=20000, Q=150, ntrain=3000, seed=17)
    c = p.ctx(T=2, sample_min=1 << 13, cand_cap=8192, prune_filter=0)
    q = torch.from_numpy(p.q).cuda()
    ws = c.alloc_workspace(150, 10, FOREST)
    ids, dist = torch.empty((150, 10), dtype=torch.int32, device="cuda"), torch.empty((150, 10), device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c.set_stream(torch.cuda.current_stream().cuda_stream)  # the capturing stream
        c.search(q, 10, FOREST, ids, dist, ws)
    c.set_stream(torch.cuda.current_stream().cuda_stream)
    for i in range(3):
        q.copy_(torch.from_numpy(np.roll(p.q, 31 * i, axis=0)))
        want = c.search(q, 10, FOREST, ws=ws)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])
