"""The matrix-core encoders at the sizes where they can go wrong: every number of 16-dimension blocks and both sides of
their edges, aligned and unaligned rows, codebooks that end inside a tile, chunks of 32 vectors and their remainders,
groups beyond 128 dimensions (the float32 matrix instruction, through LDS or streamed per lane), values that are not finite
or far from the origin.  Codes are whole numbers: exact, against the float32 oracle."""
import numpy as np
import pytest

import oracle
from workload import aligned_low_parts, near_tie_vectors

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1509_05186_amd as etf  # noqa: E402


def encoder(cb):
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    c.pq_set_codebooks(cb)
    return c


def encode(c, x):
    got = c.pq_encode_device(torch.from_numpy(x).cuda())
    torch.cuda.synchronize()
    return got.cpu().numpy()


@pytest.mark.parametrize("ds,M,K,n", [
    (1, 3, 256, 33), (6, 4, 100, 1000), (13, 4, 256, 31), (16, 8, 128, 4097), (16, 16, 256, 700), (17, 2, 129, 65),
    (25, 4, 64, 333), (32, 8, 256, 1025), (33, 2, 33, 97), (48, 5, 256, 640), (61, 1, 31, 100), (64, 3, 256, 257),
    (65, 2, 256, 95), (80, 2, 200, 160), (96, 2, 256, 64), (97, 1, 256, 129), (120, 3, 256, 300), (126, 2, 256, 40),
    (128, 2, 256, 1), (12, 1, 1, 50),
])
def test_edges_of_blocks_tiles_and_chunks(ds, M, K, n):
    print("encoder edges: ds", ds, "M", M, "K", K, "n", n, flush=True)
    rng = np.random.default_rng(ds * 1000 + M)
    cb = rng.normal(size=(M, K, ds)).astype(np.float32)
    c = encoder(cb)
    x = rng.normal(size=(n, M * ds)).astype(np.float32)
    assert np.array_equal(encode(c, x), oracle.encode_f32(x, cb))
    ties = near_tie_vectors(cb, n, seed=ds) if K > 1 else x
    assert np.array_equal(encode(c, ties), oracle.encode_f32(ties, cb))


@pytest.mark.parametrize("ds,M,K,n", [
    (129, 2, 256, 300), (130, 3, 100, 257), (131, 2, 50, 333), (132, 3, 256, 129), (132, 2, 100, 65), (160, 2, 33, 128),
    (164, 1, 256, 1), (250, 2, 200, 97), (256, 2, 256, 255), (340, 1, 7, 513),
])
@pytest.mark.parametrize("wide", [1, 0])
def test_groups_beyond_128_dimensions(ds, M, K, n, wide):
    """Aligned rows take the kernel through LDS with encode_wide = 1, unaligned ones and encode_wide = 0 the streaming one."""
    print("encoder, wide groups: ds", ds, "M", M, "K", K, "n", n, "encode_wide", wide, flush=True)
    rng = np.random.default_rng(ds * 1000 + M)
    cb = rng.normal(size=(M, K, ds)).astype(np.float32)
    c = encoder(cb)
    c.set_option("encode_wide", wide)
    x = rng.normal(size=(n, M * ds)).astype(np.float32)
    assert np.array_equal(encode(c, x), oracle.encode_f32(x, cb))
    ties = near_tie_vectors(cb, n, seed=ds)
    assert np.array_equal(encode(c, ties), oracle.encode_f32(ties, cb))
    far = (cb[np.arange(M)[None, :], rng.integers(0, K, (n, M))].reshape(n, M * ds) + np.float32(50)).astype(np.float32)
    assert np.array_equal(encode(c, far), oracle.encode_f32(far, cb))


def test_rows_that_are_not_aligned():
    """The same vectors at a 4-byte offset: the streaming kernel beyond 128 dimensions, single words up to there."""
    print("encoder: rows at an odd address", flush=True)
    rng = np.random.default_rng(12)
    for ds in (16, 120, 132):
        cb = rng.normal(size=(2, 256, ds)).astype(np.float32)
        x = near_tie_vectors(cb, 301, seed=ds)
        flat = torch.empty(x.size + 1, dtype=torch.float32, device="cuda")
        flat[1:] = torch.from_numpy(x.ravel()).cuda()
        got = encoder(cb).pq_encode_device(flat[1:].view(x.shape))
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), oracle.encode_f32(x, cb))


@pytest.mark.parametrize("ds", [16, 120])
def test_most_vectors_take_the_rule(ds):
    print("encoder: values far from the origin and spread codebooks, ds", ds, flush=True)
    rng = np.random.default_rng(ds)
    cb = rng.normal(size=(4, 256, ds)).astype(np.float32)
    cb[:, 1::2] = cb[:, ::2] * np.float32(1 + 2.0 ** -22)  # pairs that only the rule tells apart
    cb[2] += 300.0
    cb[3, 7] *= 1e6                                        # one codeword makes every bound loose
    c = encoder(cb)
    x = np.concatenate([cb[m][rng.integers(0, 256, 3000)] + rng.normal(size=(3000, ds)) * 0.1 for m in range(4)], 1).astype(np.float32)
    assert np.array_equal(encode(c, x), oracle.encode_f32(x, cb))


@pytest.mark.parametrize("ds", [4, 7, 8, 12, 16, 17, 20, 25, 40, 64, 96, 128])
def test_split_errors_that_point_the_same_way(ds):
    """What two bf16 numbers leave out of a value makes the farther of two codewords look the nearer one by as much as the
    split can; random values stay a factor of ten below (see tests/test_split_bounds.py for the sizes)."""
    print("encoder: aligned low parts, ds", ds, flush=True)
    made = [aligned_low_parts(ds, f) for f in (0.3, 0.6, 0.8, 0.85, 0.9, 0.95, 0.98, 0.99)]
    cb = np.stack([m[0] for m in made])
    x = np.concatenate([m[1] for m in made])[None].repeat(33, 0)
    x[1::2] = -x[1::2]                                     # the other half: ordinary vectors of the same codebooks
    want = oracle.encode_f32(x, cb)
    assert (want[::2] == 1).all()
    assert np.array_equal(encode(encoder(cb), x), want)


@pytest.mark.parametrize("ds,K", [(16, 256), (16, 40), (6, 256), (132, 256), (130, 100)])
@pytest.mark.parametrize("wide", [0, 1])
def test_values_that_are_not_finite_stay_their_own(ds, K, wide):
    """A vector without a distance below the largest float in a group gets codeword 0 there, as by the rule for every codeword;
    its other groups and the other vectors keep their codes."""
    print("encoder: NaN and infinities in some groups, ds", ds, "K", K, flush=True)
    rng = np.random.default_rng(8)
    cb = rng.normal(size=(4, K, ds)).astype(np.float32)
    c = encoder(cb)
    c.set_option("encode_wide", wide)
    x = rng.normal(size=(500, 4 * ds)).astype(np.float32)
    bad = np.zeros((500, 4), dtype=bool)
    for i, v in ((3, np.nan), (77, np.inf), (78, -np.inf), (499, 3e38)):
        x[i, ds * (i % 4) + 5] = v
        bad[i, i % 4] = True
    got = encode(c, x)
    with np.errstate(all="ignore"):
        want = oracle.encode_f32(x, cb)
    assert (want[bad] == 0).all()
    assert np.array_equal(got, want)
