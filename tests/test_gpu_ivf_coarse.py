"""The coarse distances on the bf16 matrix cores (queries and centroids as sums of two bf16 numbers, dimensions a multiple of
32): the probed cells and their order must be the float32 rule's, where the split is worst: nearly equal centroids, data
far from the origin, values of very different size, values that are not finite.  Every output bit for bit as with the rule
for every cell (option ivf_coarse_kernel = 1, which tests/test_gpu_ivf.py pins to the oracle)."""
import numpy as np
import pytest

import oracle
from workload import aligned_low_parts

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1509_05186_amd as etf  # noqa: E402


def both(cent, x, q, w, k, M=8):
    d = x.shape[1]
    cb = np.random.default_rng(1).normal(size=(M, 16, d // M)).astype(np.float32) * np.float32(np.abs(x[np.isfinite(x)]).std() * 0.1 + 1e-3)
    out = []
    for kernel in (0, 1):
        c = etf.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
        c.set_option("ivf_coarse_kernel", kernel)
        c.pq_set_codebooks(cb)
        c.ivf_set_coarse(cent)
        cells, codes = c.ivf_assign_device(torch.from_numpy(x).cuda())
        cells, codes = cells.cpu().numpy(), codes.cpu().numpy()
        c.ivf_build(cells, codes)
        c.ivf_upload()
        ids, dist = c.ivf_search(torch.from_numpy(q).cuda(), k, w)
        torch.cuda.synchronize()
        out.append((cells, codes, ids.cpu().numpy(), dist.cpu().numpy()))
    for a, b in zip(*out):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")


# queries around 128 per workgroup, cells around 256; one stage of 32 dimensions and several
@pytest.mark.parametrize("d,cells,Q", [(32, 255, 127), (64, 257, 129), (96, 1000, 1), (128, 512, 300), (960, 64, 130)])
@pytest.mark.parametrize("kind", ["plain", "near", "far", "scales"])
def test_split_products_keep_the_rules_cells(d, cells, Q, kind):
    print("split coarse distances d", d, "cells", cells, "Q", Q, kind, flush=True)
    rng = np.random.default_rng(d + cells)
    cent = rng.normal(size=(cells, d))
    if kind == "near":      # pairs of centroids a few units in the last place apart
        cent[1::2] = cent[:cells - cells % 2:2][:len(cent[1::2])] * (1 + 2.0 ** -21)
    if kind == "far":
        cent += 500.0
    if kind == "scales":
        cent *= 10.0 ** rng.uniform(-3, 3, size=(1, d))
    pick = lambda n: cent[rng.integers(0, cells, n)] + rng.normal(size=(n, d)) * 0.2 * np.abs(cent).mean(0)
    both(cent.astype(np.float32), pick(1500).astype(np.float32), pick(Q).astype(np.float32), min(cells, 16), 10)


def test_queries_that_are_not_finite():
    print("split coarse distances: NaN, infinities and the largest floats", flush=True)
    rng = np.random.default_rng(4)
    cent = rng.normal(size=(300, 32)).astype(np.float32)
    x = rng.normal(size=(900, 32)).astype(np.float32)
    q = rng.normal(size=(140, 32)).astype(np.float32)
    q[3, 4], q[77, 0], q[139, 31] = np.inf, 3.4e38, -1e25
    both(cent, x, q, 8, 5)


@pytest.mark.parametrize("d", [32, 64])
def test_split_errors_that_point_the_same_way(d):
    """The farther of two centroids looks the nearer one by as much as the split can (tests/test_split_bounds.py)."""
    print("split coarse distances: aligned low parts, d", d, flush=True)
    for fraction in (0.6, 0.9, 0.99):
        cent, x = aligned_low_parts(d, fraction)
        v = np.tile(x, (40, 1))
        v[1::2] = -x
        both(cent, v, v[:33], 1, 5)
