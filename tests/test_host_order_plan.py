"""The plan of searches that put their queries in order, from the workspace sizes that a host-only context computes."""
import numpy as np
import pytest

import paper_1509_05186_amd as etf

FOREST = etf.ETF_MODE_FOREST


def clusters(N, M=8, groups=40, seed=0):
    """Codebooks of 32 tight groups of 8 codewords, and codes around `groups` centres: one of those groups in every chunk, and a number in
    the last three, whose codewords are small, that makes the codes distinct.  M x 4 dimensions."""
    rng = np.random.default_rng(seed)
    cb = (np.repeat(rng.normal(0, 3, (M, 32, 4)), 8, axis=1) + rng.normal(0, 0.1, (M, 256, 4))).astype(np.float32)
    cb[M - 3:] *= 0.03
    centre = 8 * rng.integers(0, 32, (groups, M))[rng.integers(0, groups, N)]
    codes = (centre + rng.integers(0, 8, (N, M))).astype(np.uint8)
    i = np.arange(N)
    codes[:, M - 3], codes[:, M - 2], codes[:, M - 1] = i >> 16, (i >> 8) & 255, i & 255
    return cb, codes


def near(cb, codes, n, seed=1):
    """n queries beside vectors of the index."""
    rng = np.random.default_rng(seed)
    row = codes[rng.integers(0, len(codes), n)]
    x = cb[np.arange(cb.shape[0])[None, :], row].reshape(n, -1)
    return x + rng.normal(0, 0.05, x.shape).astype(np.float32)


def context(N, M=8, groups=40, seed=0, T=2, device=None, **opts):
    cb, codes = clusters(N, M, groups, seed)
    c = etf.Context(device=device)
    for name, v in opts.items():
        c.set_option(name, v)
    c.pq_set_codebooks(cb)
    c.index_build(codes, T=T)
    return c


def size(c, prune, Q, k):
    c.set_option("prune_filter", prune)
    return c.workspace_bytes(Q, k, FOREST)


@pytest.mark.parametrize("M", [8, 16])
def test_a_batch_s_kept_blocks_fit_32_bits(M):
    """Every sub-tile (32 queries at M = 8, 16 at M = 16) may keep every block of 64: their sum sizes the units of work."""
    N = 40000
    c = context(N, M, ws_cap_bytes=1 << 50)
    most = (2**32 - 1) // ((N + 63) // 64) // (M // 4) * 64   # queries of a batch
    assert size(c, 0, most + most // 50, 10) == size(c, 0, most, 10)
    assert size(c, 0, most // 2, 10) < size(c, 0, most, 10)


@pytest.fixture(scope="module")
def clustered():
    return context(300000)


def test_the_workspace_of_a_larger_call_holds_a_smaller_one(clustered):
    """A search takes the plain plan where the ordered one does not fit: that has to fit any workspace sized for a larger call.  With
    the same k the ordered one fits too."""
    c = clustered
    for Q in (1000, 1100, 3200, 3232, 10000):
        for k in (1, 30, 99, 100, 101, 300):
            assert size(c, 1, Q, k) >= size(c, -1, Q, k)
    assert size(c, 1, 10000, 99) > size(c, 1, 10000, 101) == size(c, -1, 10000, 101)  # (queries are put in order up to k = 100)
    for k in (10, 50, 100):
        sizes = [size(c, 1, Q, k) for Q in range(1000, 12000, 32)]
        assert sizes == sorted(sizes)
    try:
        for cap in (4 << 20, 64 << 20, 256 << 20, 1 << 30):
            c.set_option("ws_cap_bytes", cap)
            for Q in (1000, 3232, 10000):
                for k in (1, 50, 101):
                    assert size(c, 0, Q, k) >= size(c, -1, Q, k)
    finally:
        c.set_option("ws_cap_bytes", 8 << 30)


def test_the_rule_goes_by_the_batch(clustered):
    """A cap that leaves batches of fewer than 1000 queries leaves the plain plan."""
    c = clustered
    try:
        one = size(c, 1, 1024, 10)
        for cap in (one * 2, one + one // 8):
            c.set_option("ws_cap_bytes", cap)
            assert size(c, 1, 10000, 10) > size(c, -1, 10000, 10)
        for cap in (one - one // 8, one // 2, one // 8):
            c.set_option("ws_cap_bytes", cap)
            assert size(c, 1, 10000, 10) == size(c, -1, 10000, 10)
        # the pairs are the batch's too
        c.set_option("ws_cap_bytes", one * 5)
        assert size(c, 2500 * 300000, 10000, 10) > size(c, -1, 10000, 10)
        assert size(c, 9000 * 300000, 10000, 10) == size(c, -1, 10000, 10)
    finally:
        c.set_option("ws_cap_bytes", 8 << 30)


def ordered(c, prune, Q, k, mode=FOREST):
    c.set_option("prune_filter", -1)
    plain = c.workspace_bytes(Q, k, mode)
    c.set_option("prune_filter", prune)
    return c.workspace_bytes(Q, k, mode) != plain


def test_which_searches_are_put_in_order(clustered):
    """2^31 pairs, twice as many below 2048 queries, 1000 queries, 3000 encodings for each of k."""
    c, Nd = clustered, 300000
    assert ordered(c, 1 << 31, 7159, 10) and not ordered(c, 1 << 31, 7158, 10)
    assert ordered(c, 1, 1000, 10) and not ordered(c, 1, 999, 10)
    assert ordered(c, 2048 * Nd, 2048, 10) and not ordered(c, 2048 * Nd + 1, 2048, 10)
    assert ordered(c, 1000 * Nd, 2000, 10) and not ordered(c, 1000 * Nd + 1, 2000, 10) and not ordered(c, 1000 * Nd, 1999, 10)
    assert ordered(c, 1, 2048, 100) and not ordered(c, 1, 2048, 101)
    assert not ordered(c, -1, 10000, 10) and ordered(c, 0, 1, 10)
    assert not ordered(c, 0, 10000, 10, etf.ETF_MODE_FLAT)
    for name, value, default in (("metric", 1, 0), ("lds16_context", 0, 1), ("lds_blocks", 3, 0), ("lds_filter", 0, 2), ("lds_filter", 1, 2)):
        c.set_option(name, value)
        assert not ordered(c, 0, 10000, 10)
        c.set_option(name, default)


@pytest.mark.parametrize("N,yes", [((1 << 18) - 1, False), (1 << 18, True)])
def test_small_indexes_are_not(N, yes):
    assert ordered(context(N), 1, 2048, 10) == yes
    assert ordered(context(N), 0, 2048, 10)


def test_indexes_without_clusters_are_not():
    rng = np.random.default_rng(0)
    c = etf.Context(device=None)
    c.pq_set_codebooks(rng.normal(0, 1, (8, 256, 4)).astype(np.float32))
    c.index_build(rng.integers(0, 256, (300000, 8)).astype(np.uint8), T=2)
    assert not ordered(c, 1, 2048, 10) and ordered(c, 0, 2048, 10)
