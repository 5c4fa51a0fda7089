"""The device build that keeps its counts on the device, against the general path (which an image buffer of exactly the
size of the index asks for) byte for byte, samples included, and against numpy's sort: at the edges of its buckets,
chunks and tiles, for every width of key, with ties everywhere, and on an input that overruns a bucket."""
import numpy as np
import pytest

from test_gpu_build import arr, check_image, image_arrays
from test_gpu_parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1509_05186_amd as etf  # noqa: E402


def build(c, codes, ids, T, chunk_begin, image_bytes):
    image = torch.zeros(image_bytes + 256, dtype=torch.uint8, device="cuda")
    off = (-image.data_ptr()) % 256
    image = image[off:off + image_bytes]
    c.index_build_device(codes, ids=ids, T=T, chunk_begin=chunk_begin, image=image)
    torch.cuda.synchronize()
    return image


def compare(codes, ids=None, T=1, chunk_begin=None, K=256, order=None, sample_min=256, sample_scale=120, path=etf.ETF_BUILD_CHAIN, numpy=True):
    N, M = codes.shape
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    c.set_option("sample_min", sample_min)
    c.set_option("sample_scale", sample_scale)
    c.pq_set_codebooks(np.random.default_rng(M).standard_normal((M, K, 1)).astype(np.float32))   # in the image: also compared
    c.index_set_chunk_order(order)
    d_codes, d_ids = torch.from_numpy(codes).cuda(), None if ids is None else torch.from_numpy(ids).cuda()
    bound = c.index_build_device_bytes(N, T, chunk_begin)[0]
    image = build(c, d_codes, d_ids, T, chunk_begin, bound)
    assert c.last_build_path() == path
    need, stats = c.index_device_bytes(), c.index_stats()
    want_codes = codes if order is None else codes[:, order]
    if numpy:
        check_image(c, image, np.ascontiguousarray(want_codes), ids)
    general = build(c, d_codes, d_ids, T, chunk_begin, need)     # below the bound: every array's place checked on the host
    assert c.last_build_path() == (etf.ETF_BUILD_GENERAL if need < bound else path)   # (the smallest indexes are as large as their bound)
    assert c.index_device_bytes() == need and c.index_stats() == stats
    assert torch.equal(image[:need], general)
    assert not image[need:].any()                                # nothing behind the index is written


def clustered(rng, N, M, K):
    codes = rng.integers(0, K, size=(N, M)).astype(np.uint8)
    codes[:, : (M + 1) // 2] //= max(1, K // 6)
    again = rng.integers(0, N, N // 4)
    codes[again] = codes[rng.integers(0, N, N // 4)]
    return codes


@pytest.mark.parametrize("N", [1, 2, 8, 9, 63, 64, 65, 1023, 1025, 4095, 4096, 4097, 5119, 8191, 8193, 70001])
def test_sizes(N):
    say("build chain, sizes: N", N)
    rng = np.random.default_rng(N)
    compare(clustered(rng, N, 8, 256), T=2)
    compare(clustered(rng, N, 8, 256), rng.permutation(3 * N).astype(np.int32)[:N], T=1)


@pytest.mark.parametrize("M,T,chunk_begin", [
    (1, 1, None), (2, 2, None), (3, 1, None), (4, 1, None), (4, 2, None), (4, 4, None),       # keys of one word
    (5, 1, None), (7, 2, [0, 1, 7]), (8, 1, None), (8, 4, None), (8, 8, None), (8, 3, [0, 5, 6, 8]),   # two words
    (9, 1, None), (11, 2, [0, 9, 11]), (12, 3, None), (16, 1, None), (16, 2, None), (16, 4, None), (16, 5, [0, 4, 8, 12, 14, 16]), (16, 16, None), (16, 2, [0, 1, 16]),
])
@pytest.mark.parametrize("with_ids", [False, True])
def test_shapes(M, T, chunk_begin, with_ids):
    say("build chain, shapes: M", M, "T", T, chunk_begin, "ids", with_ids)
    rng = np.random.default_rng(100 * M + T)
    N, K = 20011, 200
    codes = clustered(rng, N, M, K)
    ids = np.sort(rng.integers(0, 50, N).astype(np.int32) * 1000)[::-1].copy() if with_ids else None   # equal ids: positions decide
    path = etf.ETF_BUILD_CHAIN if T <= 4 else etf.ETF_BUILD_GENERAL     # (more trees: the chain would need more workspace)
    compare(codes, ids, T, chunk_begin, K=K, order=list(rng.permutation(M)) if M in (7, 12) else None, path=path)


@pytest.mark.parametrize("N", [1 << 16, 1000003, (1 << 21) + 1, 5 << 20, 1 << 23, (1 << 23) + 1])
def test_workspace_is_that_of_the_general_path(N):
    say("build chain: workspace for N", N)
    c = etf.Context(device=0)
    want = None
    for M, T, chunk_begin in [(4, 1, None), (4, 4, None), (8, 2, None), (8, 3, [0, 5, 6, 8]), (8, 4, None), (8, 8, None), (16, 1, None),
                              (16, 2, [0, 1, 16]), (16, 4, None), (16, 5, [0, 4, 8, 12, 14, 16]), (16, 16, None)]:
        c.pq_set_codebooks(np.zeros((M, 256, 1), dtype=np.float32))
        got = c.index_build_device_bytes(N, T, chunk_begin)[1]
        want = want or got
        assert got == want and got <= 70 * N, (M, T)      # (the general path's does not depend on the shape)


@pytest.mark.parametrize("kind", ["equal", "sorted", "descending", "two", "last_byte"])
def test_orders_and_ties(kind):
    say("build chain, input", kind)
    rng = np.random.default_rng(3)
    N, M = 50003, 8
    codes = rng.integers(0, 256, size=(N, M)).astype(np.uint8)
    if kind == "equal":
        codes[:] = 7                                             # one encoding in every bucket
    elif kind == "two":
        codes[:] = 255
        codes[N // 3] = 0
    elif kind == "last_byte":
        codes[:, :-1] = 255                                      # keys that differ in the last byte only, the largest among them
    else:
        codes = codes[np.lexsort(codes.T[::-1])]
        if kind == "descending":
            codes = codes[::-1].copy()
    compare(codes, T=2)
    compare(codes, T=1)


def mix64(z):
    m = (1 << 64) - 1
    z = (z + 0x9E3779B97F4A7C15) & m
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
    return z ^ (z >> 31)


def overrunning_codes():
    """Samples that say nothing about the rest, so that one bucket takes nearly all."""
    rng = np.random.default_rng(9)
    N, M = 40000, 8
    codes = rng.integers(1, 256, size=(N, M)).astype(np.uint8)
    s = np.arange(N >> 7)
    codes[s * 128 + np.array([mix64(0x2545F4914F6CDD1D ^ int(i)) & 127 for i in s])] = 0
    return codes


def test_bucket_overrun():
    say("build chain: a bucket of the vectors runs over")
    compare(overrunning_codes(), T=2, path=etf.ETF_BUILD_GENERAL_AFTER_CHAIN)


def build_in_place(codes, ids, T, order, at):
    """The index of codes and ids that lie in the image itself, each at the given array's place."""
    N, M = codes.shape
    out = []
    for inside in (False, True):
        c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
        c.pq_set_codebooks(np.zeros((M, 256, 1), dtype=np.float32))
        c.index_set_chunk_order(order)
        image = torch.zeros(c.index_build_device_bytes(N, T)[0] + 256, dtype=torch.uint8, device="cuda")
        off = (-image.data_ptr()) % 256
        image = image[off:image.numel() - 256 + off]
        given = {"codes": torch.from_numpy(codes).cuda(), "ids": None if ids is None else torch.from_numpy(ids).cuda()}
        if inside:
            for name, array in at.items():
                x = given[name]
                place = image[getattr(lay, array):][:x.numel() * x.element_size()]
                place.copy_(x.reshape(-1).view(torch.uint8))
                given[name] = place.view(x.dtype).view(x.shape)
        c.index_build_device(given["codes"], ids=given["ids"], T=T, image=image)
        torch.cuda.synchronize()
        lay = c.index_layout()
        out.append((c, image))
    return out


def assert_same_arrays(out, M):
    (a, ia), (b, ib) = out
    assert a.index_stats() == b.index_stats()
    for name, off, nbytes in image_arrays(a.index_layout(), a.index_stats(), M):
        assert torch.equal(ia[off:off + nbytes], ib[off:off + nbytes]), name


@pytest.mark.parametrize("T", [1, 2])
@pytest.mark.parametrize("with_ids", [False, True])
def test_bucket_overrun_of_codes_in_the_image(T, with_ids):
    say("build chain: codes (and ids) at their place in the image, another chunk order, a bucket that runs over: T", T, "ids", with_ids)
    codes = overrunning_codes()
    ids = np.random.default_rng(11).permutation(3 * len(codes)).astype(np.int32)[:len(codes)] if with_ids else None
    at = {"codes": "codes", "ids": "ids_in"} if with_ids else {"codes": "codes"}
    out = build_in_place(codes, ids, T, [3, 1, 7, 0, 2, 6, 4, 5], at)
    assert all(c.last_build_path() == etf.ETF_BUILD_GENERAL_AFTER_CHAIN for c, _ in out)
    assert_same_arrays(out, codes.shape[1])


@pytest.mark.parametrize("at,path", [
    ({"codes": "codes"}, etf.ETF_BUILD_CHAIN),
    ({"codes": "codes", "ids": "ids_in"}, etf.ETF_BUILD_CHAIN),
    ({"codes": "ids_in"}, etf.ETF_BUILD_GENERAL),        # over an array that the first kernel writes
    ({"codes": "ids_sorted"}, etf.ETF_BUILD_CHAIN),      # ... and one that only later ones do
    ({"ids": "ids_sorted"}, etf.ETF_BUILD_CHAIN),
])
def test_inputs_in_the_image(at, path):
    say("build chain: inputs that lie in the image:", at)
    rng = np.random.default_rng(13)
    N = 300007
    codes = rng.integers(0, 256, size=(N, 8)).astype(np.uint8)
    out = build_in_place(codes, rng.permutation(N).astype(np.int32) if "ids" in at else None, 2, None, at)
    assert out[0][0].last_build_path() == etf.ETF_BUILD_CHAIN and out[1][0].last_build_path() == path
    assert_same_arrays(out, 8)


@pytest.mark.parametrize("M,T", [(8, 2), (16, 4)])
def test_bucket_overrun_in_a_tree(M, T):
    say("build chain: the vectors' buckets hold, those of the last tree do not: M", M, "T", T)
    rng = np.random.default_rng(10)
    N, D = 40000, M // T
    codes = rng.integers(1, 256, size=(N, M)).astype(np.uint8)
    codes[:, :4] = np.arange(N, dtype=">u4").view(np.uint8).reshape(N, 4)   # all distinct: encoding e is row e
    s = np.arange(N >> 7)
    codes[s * 128 + np.array([mix64(0x2545F4914F6CDD1D ^ int(i)) & 127 for i in s]), M - D:] = 0
    codes = codes[rng.permutation(N)]                              # the vectors' samples are rows like any others
    compare(codes, T=1)
    compare(codes, T=T, path=etf.ETF_BUILD_GENERAL_AFTER_CHAIN)


@pytest.mark.parametrize("sample_min,sample_scale,path", [
    (1, 0, etf.ETF_BUILD_CHAIN),
    (1 << 40, 120, etf.ETF_BUILD_CHAIN),                 # every vector, every encoding
    (1, 1 << 40, etf.ETF_BUILD_CHAIN),
    (256, 1 << 62, etf.ETF_BUILD_GENERAL),               # (times a root: no 64-bit integer)
])
def test_sample_sizes(sample_min, sample_scale, path):
    say("build chain: sample_min", sample_min, "sample_scale", sample_scale)
    compare(clustered(np.random.default_rng(14), 9001, 8, 256), T=2, sample_min=sample_min, sample_scale=sample_scale, path=path)


def test_wide_buckets():
    say("build chain: more than two million vectors")
    rng = np.random.default_rng(12)
    N = (1 << 21) + 4099
    compare(clustered(rng, N, 8, 256), T=2, sample_min=32768)


@pytest.mark.parametrize("N,M,T,with_ids,path", [
    ((1 << 21) + 4099, 4, 2, False, etf.ETF_BUILD_CHAIN),       # wide buckets of the other widths of key, and with ids
    ((1 << 21) + 4099, 4, 4, True, etf.ETF_BUILD_CHAIN),
    ((1 << 21) + 4099, 8, 2, True, etf.ETF_BUILD_CHAIN),
    (1 << 23, 8, 4, True, etf.ETF_BUILD_CHAIN),                 # the largest of the chain's, and the first that are not
    ((1 << 23) + 1, 8, 2, False, etf.ETF_BUILD_GENERAL),
    (5 << 20, 16, 4, True, etf.ETF_BUILD_CHAIN),
    (5 << 20, 16, 1, False, etf.ETF_BUILD_CHAIN),
    ((5 << 20) + 1, 16, 2, True, etf.ETF_BUILD_GENERAL),
])
def test_large_builds(N, M, T, with_ids, path):
    say("build chain, large: N", N, "M", M, "T", T, "ids", with_ids)
    rng = np.random.default_rng(N % 1009 + M)
    codes = clustered(rng, N, M, 256)
    ids = rng.permutation(N).astype(np.int32) if with_ids else None
    compare(codes, ids, T=T, sample_min=32768, path=path, numpy=False)


def test_other_codebooks_on_the_same_context():
    say("build chain: codebooks set again between builds of one context, also of another shape")
    rng = np.random.default_rng(15)
    c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
    for M, ds in ((8, 2), (8, 2), (4, 9), (8, 33), (16, 1), (8, 2)):
        cb = rng.standard_normal((M, 256, ds)).astype(np.float32)
        codes = torch.from_numpy(rng.integers(0, 256, size=(3001, M)).astype(np.uint8)).cuda()
        c.pq_set_codebooks(cb)
        bound = c.index_build_device_bytes(3001, 2)[0]
        image = build(c, codes, None, 2, None, bound)
        assert c.last_build_path() == etf.ETF_BUILD_CHAIN
        fresh = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
        fresh.pq_set_codebooks(cb)
        general = build(fresh, codes, None, 2, None, c.index_device_bytes())
        assert fresh.last_build_path() == etf.ETF_BUILD_GENERAL
        assert torch.equal(image[:general.numel()], general)
        assert np.array_equal(arr(image, c.index_layout().codebooks, cb.size, np.float32), cb.reshape(-1))
