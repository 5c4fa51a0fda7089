"""The plan of searches that put their queries in order, from the workspace sizes that a host-only context computes."""
import numpy as np
import pytest

import paper_1509_05186_amd as etf

FOREST = etf.ETF_MODE_FOREST


def context(N, M=8, groups=40, seed=0, T=2, d=None, **opts):
    """Codes around `groups` centres: a few neighbouring codewords in every chunk, and a number in the last three that makes them distinct."""
    rng = np.random.default_rng(seed)
    d = d or 4 * M
    centre = rng.integers(0, 248, (groups, M))[rng.integers(0, groups, N)]
    codes = (centre + rng.integers(0, 8, (N, M))).astype(np.uint8)
    i = np.arange(N)
    codes[:, M - 3], codes[:, M - 2], codes[:, M - 1] = i >> 16, (i >> 8) & 255, i & 255
    c = etf.Context(device=None)
    for name, v in opts.items():
        c.set_option(name, v)
    c.pq_set_codebooks(rng.normal(0, 1, (M, 256, d // M)).astype(np.float32))
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
