"""The error of a product of float32 numbers that go in as sums of two bf16 numbers each, x_l c_h + x_h c_l + x_h c_h, and the
decisions taken from such products: the arithmetic of the matrix-core encoder and of the inverted file's coarse distances, copied
in numpy.  bf16 has 8 significant bits: |a - a_h| <= 2^-8 |a|, what both parts leave out is at most 2^-17 |a|, and a product lacks
x_l c_l and two such rests, 2^-16 + 2 2^-17 = 2^-15 of |x c|."""
import numpy as np
import pytest

import oracle
from workload import aligned_low_parts

UNIT = 2.0 ** -24


def bf16(a):
    bits = np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)
    return ((bits + ((bits >> 16) & 1) + 0x7FFF) & np.uint32(0xFFFF0000)).view(np.float32)


def split(a):
    h = bf16(a)
    return h, bf16(a - h)


def test_what_two_bf16_numbers_leave_out():
    a = np.linspace(1, 2, 1 << 20, dtype=np.float32)
    h, low = split(a)
    assert 0.99 * 2.0 ** -8 < (np.abs(a - h) / a).max() <= 2.0 ** -8
    rest = np.abs(a.astype(np.float64) - h - low) / a
    assert 0.99 * 2.0 ** -17 < rest.max() <= 2.0 ** -17


def values(cb, x):
    """x.c - ||c||^2 / 2 of all codewords relative to the mean of 16 of them, the small products first, and ||x||^2 + max ||c||^2."""
    K, ds = cb.shape
    mu = np.zeros(ds, dtype=np.float32)
    for i in range(16):
        mu += cb[i * K >> 4]
    mu *= np.float32(0.0625)
    c, v = cb - mu, x - mu
    (ch, cl), (vh, vl) = split(c), split(v)
    acc = np.zeros(K, dtype=np.float32)
    for j in range(ds):
        acc = (acc + cl[:, j] * vh[j]) + ch[:, j] * vl[j]
    for j in range(ds):
        acc = acc + ch[:, j] * vh[j]
    norm = np.zeros(K, dtype=np.float32)
    for j in range(ds):
        norm += c[:, j] * c[:, j]
    exact = (c.astype(np.float64) * v).sum(1) - 0.5 * (c.astype(np.float64) ** 2).sum(1)
    S = (v.astype(np.float64) ** 2).sum() + float(norm.max())
    return acc - np.float32(0.5) * norm, exact, S


@pytest.mark.parametrize("ds", [4, 8, 12, 16, 20, 25, 64, 96, 128])
def test_encoder_keeps_the_nearest_codeword_in_question(ds):
    missed = 0
    for fraction in (0.5, 0.85, 0.9, 0.95, 0.99):
        cb, x = aligned_low_parts(ds, fraction)
        got, exact, S = values(cb, x)
        want = int(oracle.encode_f32(x[None], cb[None])[0, 0])
        assert want == 1
        # 256 units for the split, 1.5 ds + 8 for every other rounding of a value (2.5 ds + 8 with the blocks in two halves)
        assert np.abs(got - exact).max() <= (256 + 1.5 * ds + 8) * UNIT * S
        assert got[want] >= got.max() - ((6 if ds <= 64 else 8) * ds + 544) * UNIT * S
        missed += got[want] < got.max() - (6 * ds + 224) * UNIT * S  # what a unit roundoff of 2^-9 would allow
    assert missed > 0 or ds > 20


@pytest.mark.parametrize("d", [32, 64, 128])
def test_coarse_distances_stay_within_their_bound(d):
    """||c||^2 - 2 q.c against the rule's distance, in units of 2^-24 (||q|| + ||c||)^2: within 8 d + 16 + 272."""
    cb, x = aligned_low_parts(d, 0.9)
    (ch, cl), (xh, xl) = split(cb), split(x)
    acc = np.zeros(len(cb), dtype=np.float32)
    for j0 in range(0, d, 16):
        for a, b in ((cl, xh), (ch, xl), (ch, xh)):
            for j in range(j0, j0 + 16):
                acc = acc + a[:, j] * b[j]
    norm = (cb.astype(np.float64) ** 2).sum(1).astype(np.float32)
    got = norm - np.float32(2) * acc
    rule = np.zeros(len(cb), dtype=np.float32)
    for j in range(d):
        t = x[j] - cb[:, j]
        rule += t * t
    xx = (x.astype(np.float64) ** 2).sum()
    S = (np.sqrt(xx) + np.sqrt(norm.max())) ** 2
    off = np.abs(got.astype(np.float64) + xx - rule).max() / (UNIT * S)
    assert 128 < off <= 8 * d + 16 + 272
