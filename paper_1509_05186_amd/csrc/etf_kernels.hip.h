// HIP kernels for gfx950 (wave64).  Included only by etf_device.hip.
//
// Data layout shared by all kernels.  Queries are processed in tiles of QT = 64: lane q of a wave
// owns query q of the tile.  Every per-node quantity is a *row* of 64 floats (256 bytes), so a wave
// reads or writes one row with one fully coalesced instruction:
//   lutT   [tile][M][K][64]    transposed lookup tables: row (m, c) holds LUT[q][m][c] for the 64 queries
//   part   [tile][nodes][64]   partial sums of the internal nodes of one tree level
//   leafp  [tile][leaves][64]  per-tree result table: one row per leaf (distinct sub-encoding)
// Kernels that keep several table slices in LDS split a tile into G sub-tiles of Qs = 64 / G queries;
// a wave then works on G nodes at a time (lane = g * Qs + q).
#pragma once

#include <type_traits>

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "etf_internal.h"

namespace etf {

constexpr int WAVE = 64;
#ifndef ETF_UB
#define ETF_UB 8
#endif
constexpr int UB = ETF_UB;  // rows a wave keeps in flight

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

typedef __amdgpu_buffer_rsrc_t rsrc_t;

// raw buffer over `bytes` bytes at p (gfx9 family descriptor word 3: 32-bit data format); loads beyond
// the end return zero instead of faulting
__device__ __forceinline__ rsrc_t make_rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float buf_load(rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ void buf_store(float v, rsrc_t r, int voff, int soff)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), r, voff, soff, 0);
}


__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Runs of equal row indices.  Consecutive nodes usually share their parent row (siblings are adjacent in
// every level array), and a second load of a row that is still in flight is not served by the L1 but
// travels to the L2 again, which costs about as much as a fresh row.  So only the first entry of a run
// loads its row; the others load row 0 of the same table (resident in L1 after its first use) and take
// the value of their predecessor.  Everything is arithmetic on masks: a select or a branch between the
// loads would make the compiler split the batch and wait for each load before issuing the next.
// Lane i of a 64-entry chunk holds index my_idx; the result is 0 where entry i repeats entry i-1 (entry
// 0 is compared with the last index of the previous chunk) and ~0 where it starts a new run.
__device__ __forceinline__ uint32_t run_mask(uint32_t my_idx, int lane, int cnt, uint32_t carry_idx)
{
    const uint32_t up = (uint32_t)__shfl_up((int)my_idx, 1);
    const uint32_t before = lane == 0 ? carry_idx : up;
    return (lane < cnt && my_idx != before) ? 0xFFFFFFFFu : 0u;
}

// value of entry u: its own load where it starts a run (m = ~0), else the predecessor's value
__device__ __forceinline__ float run_pick(float loaded, float before, uint32_t m)
{
    return __uint_as_float((__float_as_uint(loaded) & m) | (__float_as_uint(before) & ~m));
}

// Position m of the index's encodings holds chunk src[m] of the encodings as the quantiser produces them (the
// builder's chunk order): slice m of a tile's tables is the table of dimension group src[m].
struct ChunkOrder {
    uint8_t src[ETF_MAX_M];
};

// ------------------------------------------------------------------------------------------------
// S1  lookup tables (paper Eq. 1, first term on each group's own dimensions), plain float32 form.
//     IP: the scalar products q_m . c instead (the paper's remark that the tables may hold scalar products).
//     grid (tiles, M), block 256: wave w computes codewords [64w, 64w+64) for the tile's 64 queries.
// ------------------------------------------------------------------------------------------------
template <bool IP>
__global__ __launch_bounds__(256) void k_lut_direct(const float *__restrict__ queries, int64_t Q, int64_t q0, int d,
                                                    int M, int K, const float *__restrict__ codebooks,
                                                    float *__restrict__ lutT, float *__restrict__ lut_public, ChunkOrder ord)
{
    const int tile = blockIdx.x, m = blockIdx.y, ms = ord.src[m];
    const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    const int ds = d / M;
    const int64_t q = q0 + (int64_t)tile * QT + lane;
    const bool live = q < Q;
    const float *qv = queries + (live ? q : 0) * d + (int64_t)ms * ds;
    const int kbase = w * 64;
    float acc[64];
#pragma unroll
    for (int i = 0; i < 64; ++i) acc[i] = 0.f;
    for (int j0 = 0; j0 < ds; j0 += 4) {
        float x[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) x[jj] = (live && j0 + jj < ds) ? qv[j0 + jj] : 0.f;
        const int nj = min(4, ds - j0);
#pragma unroll
        for (int i = 0; i < 64; ++i) {
            const int k = kbase + i;
            if (k < K) {
                const float *c = codebooks + ((int64_t)ms * K + k) * ds + j0;
                for (int jj = 0; jj < nj; ++jj) {
                    if (IP) {
                        acc[i] = fmaf(x[jj], c[jj], acc[i]);
                    } else {
                        float t = x[jj] - c[jj];
                        acc[i] = fmaf(t, t, acc[i]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 64; ++i) {
        const int k = kbase + i;
        if (k < K) {
            if (lutT) lutT[(((int64_t)tile * M + m) * K + k) * QT + lane] = acc[i];
            if (lut_public && live) lut_public[(q * M + ms) * K + k] = acc[i];
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Scalar-product searches.  The selection kernels order candidates by the bits of non-negative floats, smallest
// first; the largest scalar products are found as the smallest values of  B(q) - q.x,  B(q) = sum over groups of
// the group's largest table entry.  This kernel rewrites a tile's tables of products p[m][k] as B_m - p[m][k]
// (never negative: B_m is the maximum of the same rounded values) and stores the B_m, whose sum in group order
// (product_shift) is what the selection kernels subtract from again when they write the results.
//     A wave holds its 64 entries of every query's column in registers: one read and one write of the tables, all
//     loads in flight together (333 queries: two passes of one load at a time took 17 us, this 4.4 us).
//     grid (tiles, M), block 256: wave w takes codewords w, w + 4, ...; lane = query of the tile; K <= 256.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_lut_shift(float *__restrict__ lutT, int M, int K, float *__restrict__ bm)
{
    __shared__ float s_b[4][QT];
    const int tile = blockIdx.x, m = blockIdx.y, lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    float *t = lutT + ((int64_t)tile * M + m) * K * QT + lane;
    float v[64];
#pragma unroll
    for (int i = 0; i < 64; ++i) v[i] = t[(int64_t)min(w + 4 * i, K - 1) * QT];
    float b = v[0];
#pragma unroll
    for (int i = 1; i < 64; ++i) b = fmaxf(b, v[i]);
    s_b[w][lane] = b;
    __syncthreads();
    b = fmaxf(fmaxf(s_b[0][lane], s_b[1][lane]), fmaxf(s_b[2][lane], s_b[3][lane]));
#pragma unroll
    for (int i = 0; i < 64; ++i)
        if (w + 4 * i < K) t[(int64_t)(w + 4 * i) * QT] = b - v[i];
    if (w == 0) bm[((int64_t)tile * M + m) * QT + lane] = b;
}

// B(q) of query ql of the batch from the M maxima, added in group order
__device__ __forceinline__ float product_shift(const float *__restrict__ bm, int M, int64_t ql)
{
    const float *p = bm + (ql / QT) * M * QT + (ql % QT);
    float b = 0.f;
    for (int m = 0; m < M; ++m) b += p[(int64_t)m * QT];
    return b;
}

// ------------------------------------------------------------------------------------------------
// S1 on the matrix cores.  The table of one (tile, group) is a 256 x 64 block of squared distances
//     between K codewords and 64 queries over ds dimensions:  ||q' - c'||^2 = ||q'||^2 + ||c'||^2 - 2 c'.q'
//     with both sides shifted by the group's mean codeword.  The cross term is the dense contraction:
//     v_mfma_f32_32x32x2_f32 with A = codewords (32 rows) and B = queries (32 columns), float32 in,
//     float32 accumulate.  A wave owns 32 RB codewords x 64 queries = RB x 2 accumulator blocks.
//     Operand layout of the instruction (lane l): A[i = l % 32][k = l / 32], B[k = l / 32][j = l % 32];
//     accumulator register r of lane l is D[i = 8 * (r / 4) + 4 * (l / 32) + r % 4][j = l % 32], so for a
//     fixed r the lanes 0..31 hold 32 consecutive queries of one codeword: a 128-byte piece of a table row.
//     Entries that are small against the norms are recomputed exactly (see below).
//     IP: the tables hold the scalar products q_m . c themselves: the contraction on the unshifted vectors.
//     PUB (with IP): only lut_public is written, [q][M][K].  The operands change places, so that the lanes of a result
//     register hold 32 codewords of one query, 128 bytes of a row (the lanes' queries lie M K floats apart:
//     a store instruction was 64 pieces of 4 bytes; the tables of 10 000 queries, 8 KB each, 0.10 -> 0.03 ms).
//     RB = 2: grid (tiles, M), block 256 (wave w: codewords 64w .. 64w+63).  RB = 1 (the default launch): grid
//     (tiles, M, ceil(K / 32)), block 64 (one wave per workgroup, its 32 codewords given by blockIdx.z): eight times
//     the workgroups, each with an eighth of the entries to sweep and to recompute and a queue of 4 KB instead of
//     32 KB (a wave issues the sweeps' instructions one after the other: they, not the matrix instructions, are its
//     time; small batches need the workgroups to fill the chip, large ones the waves per SIMD to hide them).
// ------------------------------------------------------------------------------------------------
typedef float floatx16 __attribute__((ext_vector_type(16)));

template <bool IP, int RB, bool PUB = false>
__global__ __launch_bounds__(256) void k_lut_mfma(const float *__restrict__ queries, int64_t Q, int64_t q0, int d, int M,
                                                  int K, const float *__restrict__ cb, const float *__restrict__ cbc,
                                                  const float *__restrict__ cbnorm, const float *__restrict__ cbmean,
                                                  int dsp, float *__restrict__ lutT,
                                                  float *__restrict__ lut_public, ChunkOrder ord)
{
    const int tile = blockIdx.x, m = blockIdx.y, ms = ord.src[m];
    const int lane = threadIdx.x & 63, w = uniform(blockDim.x == 64 ? (int)blockIdx.z : (int)(threadIdx.x >> 6));
    const int ds = d / M;
    const int col = lane & 31, half = lane >> 5;
    const int kbase = w * 32 * RB;
    // B operand: the two queries this lane feeds (columns col and col + 32 of the tile)
    const float *qrow[2];
    bool qlive[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        const int64_t q = q0 + (int64_t)tile * QT + cb * 32 + col;
        qlive[cb] = q < Q;
        qrow[cb] = queries + (qlive[cb] ? q : 0) * d + (int64_t)ms * ds;
    }
    // A operand: the two codewords this lane feeds (rows col and col + 32 of the wave's 64)
    const float *crow[RB];
    bool clive[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int k = kbase + rb * 32 + col;
        clive[rb] = k < K;
        crow[rb] = IP ? cb + ((int64_t)ms * K + (clive[rb] ? k : 0)) * ds : cbc + ((int64_t)ms * K + (clive[rb] ? k : 0)) * dsp;
    }
    const float *mean = IP ? nullptr : cbmean + (int64_t)ms * ds;
    floatx16 acc[RB][2];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rb][cb][r] = 0.f;
    float qq[2] = {0.f, 0.f};
    // The contraction index may run over the dimensions in any order (the same for both operands): the instruction's
    // two k-slots (lanes 0..31 and 32..63) take the lower and the upper half of every block of 16 dimensions, so a
    // lane reads 8 consecutive floats of its rows per block (16-byte loads where the rows are aligned) and the loop
    // has an eighth of the load round trips.
    const int arow = IP ? ds : dsp;  // length of a row of the A operand (the centred codewords are zero padded to dsp)
    const bool wide = (ds & 3) == 0 && (d & 3) == 0 && (arow & 3) == 0 && (reinterpret_cast<uintptr_t>(queries) & 15) == 0 &&
                      (reinterpret_cast<uintptr_t>(IP ? cb : cbc) & 15) == 0 && (IP || (reinterpret_cast<uintptr_t>(cbmean) & 15) == 0);
    auto load8 = [&](const float *row, bool live, int j, int len, float (&o)[8]) {
        if (wide && live && j + 8 <= len) {
            const float4 lo = *reinterpret_cast<const float4 *>(row + j), hi = *reinterpret_cast<const float4 *>(row + j + 4);
            o[0] = lo.x; o[1] = lo.y; o[2] = lo.z; o[3] = lo.w;
            o[4] = hi.x; o[5] = hi.y; o[6] = hi.z; o[7] = hi.w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = (live && j + i < len) ? row[j + i] : 0.f;
        }
    };
    for (int j0 = 0; j0 < ds; j0 += 16) {
        const int j = j0 + 8 * half;
        float a[RB][8], b[2][8], mu[8];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) load8(crow[rb], clive[rb], j, arow, a[rb]);
        if (!IP) load8(mean, true, j, ds, mu);
#pragma unroll
        for (int cb2 = 0; cb2 < 2; ++cb2) {
            load8(qrow[cb2], qlive[cb2], j, ds, b[cb2]);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (!IP) b[cb2][i] = (qlive[cb2] && j + i < ds) ? b[cb2][i] - mu[i] : 0.f;
                qq[cb2] = fmaf(b[cb2][i], b[cb2][i], qq[cb2]);
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb2 = 0; cb2 < 2; ++cb2)
                    acc[rb][cb2] = PUB ? __builtin_amdgcn_mfma_f32_32x32x2f32(b[cb2][i], a[rb][i], acc[rb][cb2], 0, 0, 0)
                                       : __builtin_amdgcn_mfma_f32_32x32x2f32(a[rb][i], b[cb2][i], acc[rb][cb2], 0, 0, 0);
    }
    if constexpr (PUB) {
#pragma unroll
        for (int cb2 = 0; cb2 < 2; ++cb2)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t q = q0 + (int64_t)tile * QT + cb2 * 32 + 8 * (r / 4) + 4 * half + (r % 4);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const int k = kbase + rb * 32 + col;
                    if (q < Q && k < K) lut_public[(q * M + ms) * K + k] = acc[rb][cb2][r];
                }
            }
        return;
    }
    // the two halves of the wave summed the even and the odd dimensions of the same query
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) qq[cb] += __shfl_xor(qq[cb], 32);
    // The expanded form loses about 2^-23 (||q'||^2 + ||c'||^2) absolutely, which is too much for an entry
    // that is small against the norms (a codeword next to the query).  Such entries are not written here but
    // queued, and recomputed below as plain sums of (q - c)^2 by all threads of the workgroup.
    __shared__ uint16_t fix[RB == 2 ? QT * 256 : QT * 32];  // every entry of the workgroup could be small: 256 or 32 codewords x 64 queries
    __shared__ int nfix;
    // the codewords' norms from LDS: a global load per entry inside the loop below, each followed by a ballot and
    // a branch, is a chain of 32 memory latencies per lane
    __shared__ float s_cc[256];
    if (threadIdx.x == 0) nfix = 0;
    if (!IP)
        for (int k = threadIdx.x; k < K; k += blockDim.x) s_cc[k] = cbnorm[(int64_t)ms * K + k];
    __syncthreads();
    // Small entries are queued with one reservation per wave: a first sweep over the 64 values of a lane only counts
    // them (ballots, no memory), then one atomic reserves the wave's stretch of the queue and the second sweep hands
    // out the slots in order (an atomic with return per value was a chain of 64 LDS round trips: 20 us for a
    // workgroup of one wave).
    // (the norms of this lane's codewords once, in registers: a read inside the sweeps below is an LDS round trip per
    // value, and a workgroup of one wave has nothing else to run meanwhile)
    float ccv[RB][16];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) ccv[rb][r] = IP ? 0.f : s_cc[min(kbase + rb * 32 + 8 * (r / 4) + 4 * half + (r % 4), K - 1)];
    auto value = [&](int rb, int r, int cb, float &nn) -> float {
        nn = qq[cb] + ccv[rb][r];
        return IP ? acc[rb][cb][r] : nn - 2.f * acc[rb][cb][r];
    };
    int wave_small = 0;
    if (!IP) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = kbase + rb * 32 + 8 * (r / 4) + 4 * half + (r % 4);
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    float nn;
                    const float v = value(rb, r, cb, nn);
                    wave_small += __popcll(__ballot(k < K && v < 0.25f * nn));
                }
            }
    }
    int slot = 0;
    if (wave_small > 0) {
        if (lane == 0) slot = atomicAdd(&nfix, wave_small);
        slot = __builtin_amdgcn_readfirstlane(slot);
    }
    // this lane's entries of the transposed tables: row kbase + 4 half of the (tile, group), column col; every entry
    // of the sweep is a constant number of rows and columns further
    float *trow = lutT ? lutT + (((int64_t)tile * M + m) * K + kbase + 4 * half) * QT + col : nullptr;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int krel = rb * 32 + 8 * (r / 4) + (r % 4);
            const int k = kbase + 4 * half + krel;
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                float nn;
                const float v = value(rb, r, cb, nn);
                const int ql = cb * 32 + col;
                const bool small = !IP && k < K && v < 0.25f * nn;   // scalar products: the contraction is the result
                const uint64_t smask = __ballot(small);
                if (small)
                    fix[slot + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(smask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)smask, 0u))] =
                        (uint16_t)((ql << 8) | k);
                slot += __popcll(smask);
                if (!small && k < K) {
                    if (lutT) trow[krel * QT + cb * 32] = v;
                    const int64_t q = q0 + (int64_t)tile * QT + ql;
                    if (lut_public && q < Q) lut_public[(q * M + ms) * K + k] = v;
                }
            }
        }
    __syncthreads();
    const int todo = nfix;
    for (int i = threadIdx.x; i < todo; i += blockDim.x) {
        const int ql = fix[i] >> 8, k = fix[i] & 255;
        const int64_t q = q0 + (int64_t)tile * QT + ql;
        const bool live = q < Q;
        const float *x = queries + (live ? q : 0) * d + (int64_t)ms * ds;
        const float *c = cb + ((int64_t)ms * K + k) * ds;
        float sum = 0.f;
        if ((ds & 3) == 0 && (d & 3) == 0) {  // rows of both arrays are 16-byte aligned: four terms per load
            const float4 *x4 = reinterpret_cast<const float4 *>(x), *c4 = reinterpret_cast<const float4 *>(c);
#pragma unroll 4
            for (int j = 0; j < (ds >> 2); ++j) {
                float4 xv = x4[j];
                const float4 cv = c4[j];
                if (!live) xv = make_float4(0.f, 0.f, 0.f, 0.f);
                float t = xv.x - cv.x;
                sum = fmaf(t, t, sum);
                t = xv.y - cv.y;
                sum = fmaf(t, t, sum);
                t = xv.z - cv.z;
                sum = fmaf(t, t, sum);
                t = xv.w - cv.w;
                sum = fmaf(t, t, sum);
            }
        } else {
#pragma unroll 8
            for (int j = 0; j < ds; ++j) {  // unrolled so that the loads of several terms are in flight together
                const float t = (live ? x[j] : 0.f) - c[j];
                sum = fmaf(t, t, sum);
            }
        }
        if (lutT) lutT[(((int64_t)tile * M + m) * K + k) * QT + ql] = sum;
        if (lut_public && live) lut_public[(q * M + ms) * K + k] = sum;
    }
}

// ------------------------------------------------------------------------------------------------
// S2  one internal level of one tree:  part[l][i] = part[l-1][parent[i]] + LUT row (m, code[i]).
//     grid (blocks, tiles), block 256; every wave takes `per_wave` consecutive nodes.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_level(const uint8_t *__restrict__ icode, const uint32_t *__restrict__ iparent,
                                               int64_t n, const float *__restrict__ prev, int64_t nprev,
                                               float *__restrict__ out, const float *__restrict__ lutT, int M, int K,
                                               int m, int per_wave)
{
    const int tile = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int64_t wv = (int64_t)blockIdx.x * 4 + uniform(threadIdx.x >> 6);
    const int64_t lo = wv * per_wave;
    const int64_t hi = min(n, lo + per_wave);
    const float *lrow = lutT + ((int64_t)tile * M + m) * K * QT + lane;
    const float *prow = prev ? prev + (int64_t)tile * nprev * QT + lane : nullptr;
    float *orow = out + (int64_t)tile * n * QT + lane;
    // 64 nodes at a time: lane i fetches the record of node base+i, then the wave walks the nodes with
    // the record broadcast from that lane, UB row loads in flight before the first store
    float carry = 0.f;
    uint32_t carry_idx = NO_PARENT;
    for (int64_t base = lo; base < hi; base += 64) {
        const int cnt = (int)min<int64_t>(64, hi - base);
        const int my_code = lane < cnt ? (int)icode[base + lane] : 0;
        const uint32_t my_par = (prow && lane < cnt) ? iparent[base + lane] : 0u;
        const uint32_t my_m = prow ? run_mask(my_par, lane, cnt, carry_idx) : 0u;
        const uint32_t my_eff = my_par & my_m;
        carry_idx = (uint32_t)__builtin_amdgcn_readlane((int)my_par, cnt - 1);
        for (int s0 = 0; s0 < cnt; s0 += UB) {
            float a[UB], b[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int sidx = min(s0 + u, cnt - 1);
                a[u] = lrow[(int64_t)__builtin_amdgcn_readlane(my_code, sidx) * QT];
                b[u] = prow ? prow[(int64_t)(uint32_t)__builtin_amdgcn_readlane((int)my_eff, sidx) * QT] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int sidx = min(s0 + u, cnt - 1);
                const uint32_t m = (s0 + u < cnt) ? (uint32_t)__builtin_amdgcn_readlane((int)my_m, sidx) : 0u;
                b[u] = run_pick(b[u], u == 0 ? carry : b[u - 1], m);
            }
            carry = b[UB - 1];
#pragma unroll
            for (int u = 0; u < UB; ++u)
                if (s0 + u < cnt) orow[(base + s0 + u) * QT] = prow ? b[u] + a[u] : a[u];
        }
    }
}

// Stage `width` consecutive table slices (chunks m0 .. m0+width-1) of sub-tile g into LDS as [c][K][Qs].
template <int G>
__device__ __forceinline__ void stage_slices(float *lds, const float *__restrict__ lutT, int tile, int g, int M, int K,
                                             int m0, int width)
{
    constexpr int Qs = WAVE / G;
    const int total = width * K * Qs;
    const float *src = lutT + ((int64_t)tile * M + m0) * K * QT + g * Qs;
    for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
        const int row = idx / Qs, qq = idx % Qs;  // row = c * K + k
        lds[idx] = src[(int64_t)row * QT + qq];
    }
    __syncthreads();
}

// ------------------------------------------------------------------------------------------------
// S3  one leaf bucket of one tree (all leaves whose own chunk is at the same level, so with the same
//     postfix length):  leafp[row] = part[level-1][parent] + LUT(own chunk) + LUT(postfix chunks ...),
//     added left to right.  The bucket's `width` table slices live in LDS; lane = g*Qs + q handles
//     leaf (step*G + g) for query q of the sub-tile.
//     grid (blocks, G, tiles), block 256..1024, dynamic LDS = width*K*Qs*4 bytes.
// ------------------------------------------------------------------------------------------------
template <int G, int NDW>
__global__ void k_leaf(const uint8_t *__restrict__ lcodes, int width, const uint32_t *__restrict__ lparent,
                       const uint32_t *__restrict__ lrow, int64_t n, const float *__restrict__ prev, int64_t nprev,
                       float *__restrict__ out, int64_t U, const float *__restrict__ lutT, int M, int K, int m0,
                       int per_block)
{
    constexpr int Qs = WAVE / G;
    extern __shared__ float lds[];
    const int tile = blockIdx.z, sub = blockIdx.y;
    stage_slices<G>(lds, lutT, tile, sub, M, K, m0, width);
    const int lane = threadIdx.x & 63;
    const int lg = lane / Qs, qq = lane % Qs;
    const int w = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int64_t blo = (int64_t)blockIdx.x * per_block;
    const int64_t bhi = min(n, blo + per_block);
    const int col = sub * Qs + qq;
    const float *prow = prev ? prev + (int64_t)tile * nprev * QT + col : nullptr;
    float *orow = out + (int64_t)tile * U * QT + col;
    const uint32_t *rec = reinterpret_cast<const uint32_t *>(lcodes);
    // 64 leaves at a time: lane i fetches the record of leaf base+i; then every step handles G leaves
    // (lane group lg takes leaf s+lg), with UB parent rows in flight before the lookups start
    for (int64_t base = blo + (int64_t)w * 64; base < bhi; base += (int64_t)nw * 64) {
        const int cnt = (int)min<int64_t>(64, bhi - base);
        uint32_t my_dw[NDW];
#pragma unroll
        for (int i = 0; i < NDW; ++i) my_dw[i] = lane < cnt ? rec[(base + lane) * NDW + i] : 0u;
        const uint32_t my_par = (prow && lane < cnt) ? lparent[base + lane] : 0u;
        const uint32_t my_row = lane < cnt ? lrow[base + lane] : 0u;
        for (int s0 = 0; s0 < cnt; s0 += UB * G) {
            float acc[UB];
            uint32_t row[UB];
            uint32_t dw[UB][NDW];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int src = min(s0 + u * G + lg, cnt - 1);
                uint32_t par;
                if (G == 1) {
                    par = (uint32_t)__builtin_amdgcn_readlane((int)my_par, src);
                    row[u] = (uint32_t)__builtin_amdgcn_readlane((int)my_row, src);
#pragma unroll
                    for (int i = 0; i < NDW; ++i) dw[u][i] = (uint32_t)__builtin_amdgcn_readlane((int)my_dw[i], src);
                } else {
                    par = (uint32_t)__shfl((int)my_par, src);
                    row[u] = (uint32_t)__shfl((int)my_row, src);
#pragma unroll
                    for (int i = 0; i < NDW; ++i) dw[u][i] = (uint32_t)__shfl((int)my_dw[i], src);
                }
                acc[u] = prow ? prow[(int64_t)par * QT] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < UB; ++u) {
#pragma unroll
                for (int i = 0; i < NDW; ++i) {
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const int c = i * 4 + b;
                        if (c < width) acc[u] += lds[(c * K + ((dw[u][i] >> (8 * b)) & 255)) * Qs + qq];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < UB; ++u)
                if (s0 + u * G + lg < cnt) orow[(int64_t)row[u] * QT] = acc[u];
        }
    }
}

// ------------------------------------------------------------------------------------------------
// S3 for short leaves (own chunk plus at most one postfix chunk, W = 1 or 2): the same sum, but the
//     table rows are read straight from the transposed tables in global memory (a 64 KB slice per tile
//     and chunk, resident in L2) instead of being staged in LDS, so the kernel needs no LDS, runs at
//     full occupancy and has no staging phase.  Lane = query, one leaf per step, UB leaves in flight.
//     grid (blocks, tiles), block 256; every wave takes `per_wave` consecutive leaves.
// ------------------------------------------------------------------------------------------------
template <int W>
__global__ __launch_bounds__(256) void k_leaf_short(const uint8_t *__restrict__ lcodes, const uint32_t *__restrict__ lparent,
                                                    const uint32_t *__restrict__ lrow, int64_t n,
                                                    const float *__restrict__ prev, int64_t nprev, float *__restrict__ out,
                                                    int64_t U, const float *__restrict__ lutT, int M, int K, int m0,
                                                    int per_wave)
{
    const int tile = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int64_t wv = (int64_t)blockIdx.x * 4 + uniform(threadIdx.x >> 6);
    const int64_t lo = wv * per_wave;
    const int64_t hi = min(n, lo + per_wave);
    const float *lut0 = lutT + ((int64_t)tile * M + m0) * K * QT + lane;
    const float *prow = prev ? prev + (int64_t)tile * nprev * QT + lane : nullptr;
    float *orow = out + (int64_t)tile * U * QT + lane;
    const uint32_t *rec = reinterpret_cast<const uint32_t *>(lcodes);  // one 4-byte record per leaf
    float carry = 0.f;
    uint32_t carry_idx = NO_PARENT;
    for (int64_t base = lo; base < hi; base += 64) {
        const int cnt = (int)min<int64_t>(64, hi - base);
        const int my_dw = lane < cnt ? (int)rec[base + lane] : 0;
        const uint32_t my_par = (prow && lane < cnt) ? lparent[base + lane] : 0u;
        const int my_row = lane < cnt ? (int)lrow[base + lane] : 0;
        const uint32_t my_m = prow ? run_mask(my_par, lane, cnt, carry_idx) : 0u;
        const uint32_t my_eff = my_par & my_m;
        carry_idx = (uint32_t)__builtin_amdgcn_readlane((int)my_par, cnt - 1);
        for (int s0 = 0; s0 < cnt; s0 += UB) {
            float p[UB], v[UB][W];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int src = min(s0 + u, cnt - 1);
                const uint32_t dw = (uint32_t)__builtin_amdgcn_readlane(my_dw, src);
                p[u] = prow ? prow[(int64_t)(uint32_t)__builtin_amdgcn_readlane((int)my_eff, src) * QT] : 0.f;
#pragma unroll
                for (int c = 0; c < W; ++c) v[u][c] = lut0[((int64_t)c * K + ((dw >> (8 * c)) & 255)) * QT];
            }
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int src = min(s0 + u, cnt - 1);
                const uint32_t m = (s0 + u < cnt) ? (uint32_t)__builtin_amdgcn_readlane((int)my_m, src) : 0u;
                p[u] = run_pick(p[u], u == 0 ? carry : p[u - 1], m);
            }
            carry = p[UB - 1];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                if (s0 + u >= cnt) break;
                float acc = prow ? p[u] : 0.f;
#pragma unroll
                for (int c = 0; c < W; ++c) acc += v[u][c];
                orow[(int64_t)(uint32_t)__builtin_amdgcn_readlane(my_row, s0 + u) * QT] = acc;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// PQ encoding on the device (paper, Introduction: every dimension group is quantised separately to its nearest
//     codeword): codes[i][m] = argmin_c || x[i] group m - codeword c of group m ||^2, lowest c on ties.
//     Float32, every squared distance the sum of its terms in dimension order with one rounding per
//     operation (no fused multiply-add), so that a float32 reference can reproduce every decision.
//     One thread per vector and group, the sub-vector in registers (DSP = ds rounded up to 4, 8, ..., 128,
//     padded with zeros against zero-padded codewords, which adds exact zeros); the group's codewords in
//     LDS, KC at a time, read as broadcasts.
//     grid (ceil(n / 256), M), block 256, dynamic LDS KC*DSP*4 bytes.
// ------------------------------------------------------------------------------------------------
template <int DSP>
__global__ __launch_bounds__(256) void k_encode(const float *__restrict__ x, int64_t n, int d, int ds, int K, int M,
                                                const float *__restrict__ cb, uint8_t *__restrict__ codes, int KC)
{
    extern __shared__ float lds[];  // [KC][DSP]
    const int m = blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float xv[DSP];
    {
        const float *xi = x + (i < n ? i : 0) * d + (int64_t)m * ds;
#pragma unroll
        for (int j = 0; j < DSP; ++j) xv[j] = (j < ds && i < n) ? xi[j] : 0.f;
    }
    float bestd = 3.402823466e+38f;
    int best = 0;
    for (int k0 = 0; k0 < K; k0 += KC) {
        const int kc = min(KC, K - k0);
        __syncthreads();
        for (int idx = threadIdx.x; idx < kc * DSP; idx += 256) {
            const int k = idx / DSP, j = idx % DSP;
            lds[idx] = j < ds ? cb[((int64_t)m * K + k0 + k) * ds + j] : 0.f;
        }
        __syncthreads();
        for (int k = 0; k < kc; ++k) {
            const float *c = lds + k * DSP;
            float s = 0.f;
            {
                // every operation rounds on its own: without this the compiler contracts the product and the sum
                // into one fused multiply-add, whose result differs in the last bit often enough to change near-ties
#pragma clang fp contract(off)
#pragma unroll
                for (int j = 0; j < DSP; ++j) {  // plain operators: the pragma governs what is written here, not
                    const float t = xv[j] - c[j];  // the bodies of intrinsics defined elsewhere
                    const float p = t * t;
                    s = s + p;
                }
            }
            if (s < bestd) {
                bestd = s;
                best = k0 + k;
            }
        }
    }
    if (i < n) codes[i * M + m] = (uint8_t)best;
}

// ------------------------------------------------------------------------------------------------
// Rotation in front of the quantiser (Optimized Product Quantization, named in the paper's Related Work among the
//     quantisers the tree applies to): out[i] = R x[i], every component accumulated in double over the dimensions
//     in ascending order and rounded to float once (a product of two floats is exact in double: the fused
//     multiply-add changes nothing), the rule the host function and the reference follow bit for bit.
//     Rt is the rotation transposed ([j][r] = R[r][j]: neighbouring threads read neighbouring words).
//     grid (ceil(n / rows_per_block)), block 256, dynamic LDS rows_per_block * d * 4 bytes.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_rotate(const float *__restrict__ x, int64_t n, int d, const float *__restrict__ Rt,
                                                float *__restrict__ out, int rows_per_block)
{
    extern __shared__ float rot_xs[];  // [rows_per_block][d]
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
    const int rows = (int)min<int64_t>(rows_per_block, n - r0);
    for (int idx = threadIdx.x; idx < rows * d; idx += 256) rot_xs[idx] = x[r0 * d + idx];
    __syncthreads();
    for (int idx = threadIdx.x; idx < rows * d; idx += 256) {
        const int row = idx / d, r = idx - row * d;
        const float *xr = rot_xs + row * d;
        double acc = 0.0;
        for (int j = 0; j < d; ++j) acc += (double)Rt[(int64_t)j * d + r] * (double)xr[j];
        out[(r0 + row) * d + r] = (float)acc;
    }
}

// One term of the float32 rule: s + (x - c)^2 with every operation rounded on its own.
__device__ __forceinline__ float encode_rule_term(float s, float x, float c)
{
#pragma clang fp contract(off)
    const float t = x - c;
    const float pr = t * t;
    return s + pr;
}

// The float32 rule for one vector, evaluated by a whole wave (the near-ties of the matrix-core encoders): lane l takes
// codewords l, l + 64, l + 128, l + 192 (K <= 256), each distance the sum of its terms in dimension order; returns
// the codeword with the smallest (distance, index) in every lane, 0 where no distance is below the largest float (as k_encode).  xv: the vector's values of the group, cbm: the
// group's codewords [K][ds].  rows16: ds is a multiple of 4 and both rows are 16-byte aligned; then the four sums
// advance together on 16-byte loads, two steps in flight (one value per load and iteration is a memory latency per
// dimension and codeword: 0.1 ms for a single vector with 120 dimensions per group).
__device__ __forceinline__ int encode_rule_wave(const float *__restrict__ xv, const float *__restrict__ cbm, int ds, int K, int lane,
                                                bool rows16)
{
    float bestd = 3.402823466e+38f;
    int best = 0x7FFFFFFF;
    if (rows16) {
        float sacc[4] = {0.f, 0.f, 0.f, 0.f};
        const float *c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = cbm + (int64_t)min(lane + 64 * u, K - 1) * ds;
#pragma unroll 2
        for (int j = 0; j < ds; j += 4) {
            const float4 xq = *reinterpret_cast<const float4 *>(xv + j);
            float4 cq[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) cq[u] = *reinterpret_cast<const float4 *>(c[u] + j);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                sacc[u] = encode_rule_term(sacc[u], xq.x, cq[u].x);
                sacc[u] = encode_rule_term(sacc[u], xq.y, cq[u].y);
                sacc[u] = encode_rule_term(sacc[u], xq.z, cq[u].z);
                sacc[u] = encode_rule_term(sacc[u], xq.w, cq[u].w);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (lane + 64 * u < K && sacc[u] < bestd) {  // ascending index inside a lane: the first minimum stays
                bestd = sacc[u];
                best = lane + 64 * u;
            }
    } else {
        for (int k = lane; k < K; k += 64) {
            const float *c = cbm + (int64_t)k * ds;
            float sacc = 0.f;
            for (int j = 0; j < ds; ++j) sacc = encode_rule_term(sacc, xv[j], c[j]);
            if (sacc < bestd) {  // ascending k inside a lane: the first minimum stays
                bestd = sacc;
                best = k;
            }
        }
    }
#pragma unroll
    for (int dlt = 32; dlt > 0; dlt >>= 1) {
        const float od = __shfl_xor(bestd, dlt);
        const int ob = __shfl_xor(best, dlt);
        if (od < bestd || (od == bestd && ob < best)) {
            bestd = od;
            best = ob;
        }
    }
    return best == 0x7FFFFFFF ? 0 : best;
}

// ------------------------------------------------------------------------------------------------
// The same assignment with the distance evaluations on the matrix cores (the O(dKN) term of the paper's "Efficient
//     Encoding Tree Construction").  For every (vector, group) the 256 values  ||c||^2 - 2 x.c  come from the dense
//     contraction x.c (v_mfma_f32_32x32x2_f32, operands as in k_lut_mfma: A = codewords, B = vectors); they differ
//     from the float32 rule's squared distances (minus ||x||^2) by at most E = 8 (ds + 2) 2^-24 (||x||^2 + max ||c||^2),
//     a generous bound on the rounding of either form.  If the smallest value is more than 2 E below the second
//     smallest, its codeword is the float32 rule's winner as well; otherwise (a near-tie: a few vectors in a
//     thousand) the wave evaluates the rule itself for all K codewords of that vector, four per lane, and takes the
//     smallest (distance, index).  The codes are those of k_encode, bit for bit.
//     A wave owns 64 vectors and walks the codewords 64 at a time (2 x 2 accumulator blocks); per value it keeps the
//     two smallest and the index of the smallest.
//     grid (ceil(n / 256), M), block 256, K <= 256.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void k_encode_mfma(const float *__restrict__ x, int64_t n, int d, int ds, int K, int M,
                                                     const float *__restrict__ cb, uint8_t *__restrict__ codes)
{
    __shared__ float s_cc[256];
    __shared__ float s_ccmax;
    const int m = blockIdx.y;
    const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    const int col = lane & 31, half = lane >> 5;
    const float *cbm = cb + (int64_t)m * K * ds;
    // squared norms of the group's codewords (plain float32 sums: covered by E)
    {
        float cc = 0.f;
        if ((int)threadIdx.x < K)
            for (int j = 0; j < ds; ++j) cc = fmaf(cbm[(int64_t)threadIdx.x * ds + j], cbm[(int64_t)threadIdx.x * ds + j], cc);
        s_cc[threadIdx.x] = (int)threadIdx.x < K ? cc : 3.0e38f;
        float mx = (int)threadIdx.x < K ? cc : 0.f;
#pragma unroll
        for (int dlt = 32; dlt > 0; dlt >>= 1) mx = fmaxf(mx, __shfl_xor(mx, dlt));
        __syncthreads();
        if (threadIdx.x == 0) s_ccmax = 0.f;
        __syncthreads();
        if (lane == 0) atomicMax(reinterpret_cast<int *>(&s_ccmax), __float_as_int(mx));  // non-negative floats order like ints
        __syncthreads();
    }
    const int64_t v0 = (int64_t)blockIdx.x * 256 + w * 64;
    if (v0 >= n) return;
    // B operand: the two vectors this lane feeds (columns col and col + 32 of the wave's 64)
    const float *xrow[2];
    bool xlive[2];
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2) {
        const int64_t v = v0 + c2 * 32 + col;
        xlive[c2] = v < n;
        xrow[c2] = x + (xlive[c2] ? v : 0) * d + (int64_t)m * ds;
    }
    float v1[2] = {3.0e38f, 3.0e38f}, v2[2] = {3.0e38f, 3.0e38f}, xx[2] = {0.f, 0.f};
    int k1[2] = {0, 0};
    // The contraction index may run over the dimensions in any order, as long as it is the same for both operands:
    // the instruction's two k-slots (lanes 0..31 and 32..63) take the lower and the upper half of every block of 16
    // dimensions, so that a lane reads 8 consecutive floats of its row per block (two 16-byte loads where the rows
    // are aligned) instead of one float per instruction.
    const bool wide = (ds & 3) == 0 && (d & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0 && (reinterpret_cast<uintptr_t>(cb) & 15) == 0;
    auto load8 = [&](const float *row, bool live, int j, float (&o)[8]) {
        if (wide && live && j + 8 <= ds) {
            const float4 lo = *reinterpret_cast<const float4 *>(row + j), hi = *reinterpret_cast<const float4 *>(row + j + 4);
            o[0] = lo.x; o[1] = lo.y; o[2] = lo.z; o[3] = lo.w;
            o[4] = hi.x; o[5] = hi.y; o[6] = hi.z; o[7] = hi.w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = (live && j + i < ds) ? row[j + i] : 0.f;
        }
    };
    for (int p0 = 0; p0 < K; p0 += 64) {
        const float *crow[2];
        bool clive[2];
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
            const int k = p0 + rb * 32 + col;
            clive[rb] = k < K;
            crow[rb] = cbm + (int64_t)(clive[rb] ? k : 0) * ds;
        }
        floatx16 acc[2][2];
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[rb][c2][r] = 0.f;
        for (int j0 = 0; j0 < ds; j0 += 16) {
            const int j = j0 + 8 * half;
            float a[2][8], b[2][8];
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) load8(crow[rb], clive[rb], j, a[rb]);
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2) {
                load8(xrow[c2], xlive[c2], j, b[c2]);
                if (p0 == 0) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) xx[c2] = fmaf(b[c2][i], b[c2][i], xx[c2]);
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                    for (int c2 = 0; c2 < 2; ++c2)
                        acc[rb][c2] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[rb][i], b[c2][i], acc[rb][c2], 0, 0, 0);
        }
        // accumulator register r of lane l: codeword p0 + 32 rb + 8 (r / 4) + 4 (l / 32) + r % 4, vector l % 32 (+ 32 c2)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = p0 + rb * 32 + 8 * (r / 4) + 4 * half + (r % 4);
                const float cc = s_cc[k];  // 3e38 beyond K: never the smallest
#pragma unroll
                for (int c2 = 0; c2 < 2; ++c2) {
                    const float val = fmaf(-2.f, acc[rb][c2][r], cc);
                    k1[c2] = val < v1[c2] ? k : k1[c2];
                    v2[c2] = __builtin_amdgcn_fmed3f(val, v1[c2], v2[c2]);  // v1 <= v2: the median is the new second smallest
                    v1[c2] = fminf(val, v1[c2]);
                }
            }
    }
    // the two halves of the wave saw the even and the odd rows of the same columns
    const float ccmax = s_ccmax;
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2) {
        const float o1 = __shfl_xor(v1[c2], 32), o2 = __shfl_xor(v2[c2], 32);
        const int ok = __shfl_xor(k1[c2], 32);
        xx[c2] += __shfl_xor(xx[c2], 32);
        const float hi = fmaxf(v1[c2], o1);
        if (o1 < v1[c2] || (o1 == v1[c2] && ok < k1[c2])) k1[c2] = ok;
        v1[c2] = fminf(v1[c2], o1);
        v2[c2] = fminf(hi, fminf(v2[c2], o2));
    }
    // lanes 0..31 decide columns col and col + 32
    const float eps = 8.f * (float)(ds + 2) * 5.9604645e-8f;
    bool hard[2];
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2) {
        const float E = eps * (xx[c2] + ccmax);
        // (values so small that products are subnormal: the matrix instruction flushes them, E does not cover that)
        hard[c2] = xlive[c2] && (!(v2[c2] - v1[c2] > 2.f * E) || xx[c2] + ccmax < 1.0e-30f);
        if (half == 0 && xlive[c2] && !hard[c2]) codes[(v0 + c2 * 32 + col) * M + m] = (uint8_t)k1[c2];
    }
    // near-ties: the float32 rule itself for every codeword, the wave's lanes taking codewords lane, lane + 64, ...
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2) {
        uint64_t todo = __ballot(hard[c2] && half == 0);
        while (todo != 0ull) {
            const int src = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const int64_t v = v0 + c2 * 32 + src;
            const int best = encode_rule_wave(x + v * d + (int64_t)m * ds, cbm, ds, K, lane, wide);
            if (lane == 0) codes[v * M + m] = (uint8_t)best;
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The same assignment on the bf16 matrix cores (groups of at most 128 dimensions, any alignment; wider groups take
//     k_encode_wide or k_encode_mfma).  Only a decision is wanted, and only its rounding has to be proved harmless, so
//     every float32 value goes in as a sum of two bf16 numbers, a = a_h + a_l + r, and x.c as x_l.c_h + x_h.c_l + x_h.c_h:
//     three bf16 instructions of 32 cycles for 16 dimensions where the float32 instruction takes eight of 64.  bf16 has 8
//     significant bits, so |a_l| <= 2^-8 |a| and |r| <= 2^-17 |a|; a product lacks x_l c_l and two such rests, at most
//     2^-16 + 2 2^-17 = 2^-15 of |x c|.  Vectors and codewords are taken relative to a point mu near the group's codewords (their
//     mean, roughly), which changes no distance and makes the values, and with them every rounding, smaller.
//     For a (vector, group) the accumulators hold x.c - ||c||^2 / 2 of all codewords (largest = nearest).  -||c||^2 / 2
//     enters last, as the sum of three bf16 numbers against ones in an instruction of its own (as a starting value it
//     would take four LDS reads per tile and make every rounding one of the larger sum); the small products are first.
//     With S = ||x||^2 + max ||c||^2, sum |x c| <= S / 2, in units of 2^-24 S a value is off by at most: 256 (split), 1.03 ds
//     (sum of x_h.c_h and of the small products, one unit in the last place per product), 6 (the three norm slots), 0.5 ds
//     (the norm), 2 (x - mu, c - mu); the float32 rule's distance (halved) by ds + 2.  Two values together: less than
//     6 ds + 544 (from 6 blocks of 16 dimensions on the small products come first in either half of the blocks, for want of
//     registers: 1.03 ds more per value, 8 ds + 544).  So with E = (6 ds + 544) 2^-24 S every codeword
//     the rule might choose has a value of at least the largest minus E.  Where that is one codeword it is the code;
//     otherwise (a few vectors in a thousand) the float32 rule is evaluated for exactly those codewords (usually two),
//     pairs (vector, codeword) of a wave collected in LDS until they fill its lanes.  The codes are k_encode's, bit
//     for bit.
//     Which values are at or above a threshold takes no index per value: a lane keeps the maximum of every tile
//     of 32 codewords (over its 16 accumulator registers) and of every register (over the 8 tiles), one v_max3 per
//     value for both, and compares 8 + 16 maxima in the end; the codewords in question lie in marked tiles x
//     marked registers.  (Largest, second largest and index per value took four instructions a value and bound the
//     kernel once the products were cheap.)
//     A workgroup keeps the operands of as many groups as fit its LDS (16 KB per 16 dimensions, in instruction order)
//     and walks the vectors, 32 per wave and step, whole rows at a time where all groups fit.
//     What bounds it: vector and matrix issue together (about 350 vector instructions and 32 matrix instructions for 32
//     vectors of a group of 16 dimensions; a matrix instruction takes the issue slot of about two others), the matrix
//     cores for wide groups.  Kernel time against the float32 matrix instruction with three values tracked per codeword:
//     a million vectors, 8 groups of 16, 0.81 -> 0.27 ms; 250 001 vectors, 8 groups of 120, 1.63 -> 0.36 ms.
//     grid (vector chunks, ceil(M / gs)), block NW * 64, dynamic LDS encode_bf_lds().
// ------------------------------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
constexpr int ENC_PAIRS = 64;  // (vector, codeword) pairs a wave collects
constexpr size_t ENC_QUEUE_BYTES = 64 * 8 + 64 * 8 + ENC_PAIRS * 4;
__host__ __device__ constexpr size_t encode_bf_group_bytes(int NB) { return (size_t)NB * 16384 + 2048 + (size_t)NB * 64 + 16; }  // (the last 16: the largest norm, the turn)
__host__ __device__ constexpr size_t encode_bf_lds(int NB, int gs, int NW) { return gs * encode_bf_group_bytes(NB) + NW * ENC_QUEUE_BYTES; }

// eight float32 values as the sum of two bf16 numbers each
__device__ __forceinline__ void split_bf16(const f32x8 &v, bf16x8 &h, bf16x8 &l)
{
    typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
    h = __builtin_convertvector(v, bf16x8);
    const u32x4v b = __builtin_bit_cast(u32x4v, h);
    f32x8 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        r[2 * i] = v[2 * i] - __uint_as_float(b[i] << 16);
        r[2 * i + 1] = v[2 * i + 1] - __uint_as_float(b[i] & 0xFFFF0000u);
    }
    l = __builtin_convertvector(r, bf16x8);
}

// WIDE: rows that can be read 16 bytes at a time
template <int NB, bool WIDE, int NW>
__global__ __launch_bounds__(NW * 64, NW / 4) void k_encode_bf(const float *__restrict__ x, int64_t n, int d, int ds, int K, int M,
                                                               const float *__restrict__ cb, uint8_t *__restrict__ codes, int gs)
{
    constexpr int DSP = NB * 16, NT = NW * 64;
    constexpr int TS = 2;          // codeword tiles at a time
    constexpr bool AHEAD = NB < 6;  // registers for the next step's values (else its lines are only drawn into the cache)
    extern __shared__ __align__(16) char enc_raw[];
    const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int m0 = (int)blockIdx.y * gs, gl = min(gs, M - m0);
    bf16x8 *ops = reinterpret_cast<bf16x8 *>(enc_raw);                      // [gs][8 tiles][NB][high, low][64 lanes]
    char *behind = enc_raw + (size_t)gs * NB * 16384;
    uint64_t *hbest = reinterpret_cast<uint64_t *>(behind) + w * 64;        // per open vector: smallest (distance, codeword)
    behind += NW * 64 * 8;
    uint64_t *hvec = reinterpret_cast<uint64_t *>(behind) + w * 64;         // ... and whose it is: vector << 8 | group
    behind += NW * 64 * 8;
    uint2 *nrm = reinterpret_cast<uint2 *>(behind);                         // [gs][256]: four bf16 (the last is zero)
    behind += (size_t)gs * 2048;
    float *mu = reinterpret_cast<float *>(behind);                          // [gs][DSP]
    behind += (size_t)gs * DSP * 4;
    uint32_t *ccm = reinterpret_cast<uint32_t *>(behind);                   // [gs] largest ||c||^2 (bits)
    uint32_t *turn = ccm + gs;                                              // work handed out so far
    behind += (size_t)gs * 16;
    uint32_t *pairs = reinterpret_cast<uint32_t *>(behind) + w * ENC_PAIRS;  // slot << 8 | codeword

    // ---- the point the group is taken relative to: the mean of up to 16 codewords
    if ((int)threadIdx.x <= gl) (threadIdx.x == 0 ? turn : ccm + threadIdx.x - 1)[0] = 0u;
    for (int idx = threadIdx.x; idx < gl * DSP; idx += NT) {
        const int ml = idx / DSP, j = idx % DSP;
        float s = 0.f;
        if (j < ds) {
            const float *c = cb + (int64_t)(m0 + ml) * K * ds + j;
#pragma unroll
            for (int i = 0; i < 16; ++i) s += c[(int64_t)((i * K) >> 4) * ds];
        }
        mu[idx] = s * 0.0625f;
    }
    __syncthreads();
    // ---- codewords as operands
    const int rows = (K + 32 * TS - 1) / (32 * TS) * (32 * TS);  // of the tiles that are walked
    for (int idx = threadIdx.x; idx < gl * rows; idx += NT) {
        const int ml = idx / rows, k = idx - ml * rows;
        const float *c = cb + ((int64_t)(m0 + ml) * K + min(k, K - 1)) * ds;
        bf16x8 *dst = ops + (size_t)(ml * 8 + (k >> 5)) * NB * 128 + (k & 31);
        float cc = 0.f;
#pragma unroll 2
        for (int p = 0; p < 2 * NB; ++p) {
            f32x8 v;
            if (WIDE) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int j = 8 * p + 4 * q;
                    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (j < ds) t = *reinterpret_cast<const float4 *>(c + j);
                    v[4 * q] = t.x; v[4 * q + 1] = t.y; v[4 * q + 2] = t.z; v[4 * q + 3] = t.w;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = 8 * p + i < ds ? c[8 * p + i] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float u = mu[ml * DSP + 8 * p + i];
                v[i] = (k < K && 8 * p + i < ds) ? v[i] - u : 0.f;
                cc = fmaf(v[i], v[i], cc);
            }
            bf16x8 h, l;
            split_bf16(v, h, l);
            dst[(p >> 1) * 128 + (p & 1) * 32] = h;
            dst[(p >> 1) * 128 + 64 + (p & 1) * 32] = l;
        }
        // -||c||^2 / 2 as three bf16 numbers; far below every value beyond K
        const float h0 = k < K ? -0.5f * cc : -3.0e38f;
        const __bf16 n0 = (__bf16)h0;
        const float h1 = h0 - (float)n0;
        const __bf16 n1 = (__bf16)h1;
        const __bf16 n2 = (__bf16)(h1 - (float)n1);
        const uint32_t b0 = __builtin_bit_cast(uint16_t, n0), b1 = __builtin_bit_cast(uint16_t, n1), b2 = __builtin_bit_cast(uint16_t, n2);
        nrm[ml * 256 + k] = make_uint2(b0 | (b1 << 16), b2);
        if (k < K) atomicMax(&ccm[ml], __float_as_uint(cc) & 0x7FFFFFFFu);  // non-negative floats order like their bits, NaN above all
    }
    __syncthreads();

    const float eps = (float)((NB >= 6 ? 8 : 6) * ds + 544) * 5.9604645e-8f;
    const float inf = __uint_as_float(0x7F800000u);
    int hcount = 0, pcount = 0;
    // the float32 rule for the collected pairs, a lane each
    auto evaluate = [&]() {
        __builtin_amdgcn_wave_barrier();
        for (int i = lane; i < pcount; i += 64) {
            const uint32_t p = pairs[i];
            const int slot = (int)(p >> 8), k = (int)(p & 255u);
            if (k >= K) continue;
            const uint64_t hv = hvec[slot];
            const int m = (int)(hv & 255u);
            const float *xv = x + (int64_t)(hv >> 8) * d + (int64_t)m * ds;
            const float *c = cb + ((int64_t)m * K + k) * ds;
            float s = 0.f;
            if (WIDE) {
#pragma unroll 4
                for (int j = 0; j < ds; j += 4) {
                    const float4 xq = *reinterpret_cast<const float4 *>(xv + j), cq = *reinterpret_cast<const float4 *>(c + j);
                    s = encode_rule_term(s, xq.x, cq.x);
                    s = encode_rule_term(s, xq.y, cq.y);
                    s = encode_rule_term(s, xq.z, cq.z);
                    s = encode_rule_term(s, xq.w, cq.w);
                }
            } else {
                for (int j = 0; j < ds; ++j) s = encode_rule_term(s, xv[j], c[j]);
            }
            if (s < 3.402823466e+38f) atomicMin(reinterpret_cast<unsigned long long *>(&hbest[slot]), ((unsigned long long)__float_as_uint(s) << 32) | (uint32_t)k);
        }
        __builtin_amdgcn_wave_barrier();
        pcount = 0;
    };
    auto settle = [&]() {
        evaluate();
        if (lane < hcount) {
            const uint64_t hv = hvec[lane];
            codes[(int64_t)(hv >> 8) * M + (int64_t)(hv & 255u)] = (uint8_t)hbest[lane];
        }
        __builtin_amdgcn_wave_barrier();
        hcount = 0;
    };

    // A unit of work is a chunk of 32 vectors and up to four groups; the waves of the workgroup take the units of its
    // chunks in turn (dealt out beforehand, the last waves worked alone for a sixth of the time).
    const int64_t chunks = (n + 31) / 32;
    const int parts = (gl + 3) / 4;
    int64_t chunk = 0;
    int ml = 0, mlend = 0;
    auto take = [&]() {
        uint32_t u = 0;
        if (lane == 0) u = atomicAdd(turn, 1u);
        u = (uint32_t)uniform((int)u);
        const uint32_t i = u / (uint32_t)parts;
        ml = 4 * (int)(u - i * (uint32_t)parts);
        mlend = min(ml + 4, gl);
        chunk = blockIdx.x + (int64_t)gridDim.x * i;
    };
    // The values of a step, one step ahead: lane (col, half) has dimensions 16 nb + 8 half .. + 7 of vector col.  Through
    // a buffer over the step's rows, whose end turns what lies beyond the group (or the last vector) into zeros.
    f32x8 raw[NB];
    const uint32_t voff = (uint32_t)(col * d + 8 * half) * 4u;
    auto fetch = [&](int64_t chunk, int ml) {
        const int64_t v0 = chunk * 32;
        const rsrc_t rr = make_rsrc(x + v0 * d, (uint32_t)min<int64_t>(32, n - v0) * (uint32_t)d * 4u);
        const int so = (m0 + ml) * ds * 4;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int i = 0; i < 8; i += WIDE ? 4 : 1) {
                const int j = 16 * nb + i;
                const uint32_t vo = (nb < NB - 2 || j + 8 * half < ds) ? voff + (uint32_t)j * 4u : 0x7FFFFFFFu;
                if (WIDE) {
                    const auto t = __builtin_amdgcn_raw_buffer_load_b128(rr, (int)vo, so, 0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) raw[nb][i + q] = __uint_as_float(t[q]);
                } else {
                    raw[nb][i] = buf_load(rr, (int)vo, so);
                }
            }
    };
    // the codes of a step leave through a buffer as well: lanes without one store past its end, without a branch (behind a
    // branch the wait for the next step's values also waits for the store)
    auto put = [&](int64_t chunk, int m, bool write, uint32_t code) {
        const rsrc_t rc = make_rsrc(codes + chunk * 32 * M, (uint32_t)min<int64_t>(32, n - chunk * 32) * (uint32_t)M);
        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)code, rc, write ? col * M + m : 0x7FFFFFFF, 0, 0);
    };
    const uint32_t one = half == 0 ? 0x3F80u : 0u;  // bf16 1.0 in the lower half's first three slots
    const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(one | (one << 16), one, 0u, 0u));
    // operand of a tile's codewords; narrow groups have registers to read those of the next tiles ahead
    auto operand = [&](int g, int tile, int nb, int low) -> bf16x8 { return ops[((g * 8 + tile) * NB + nb) * 128 + low * 64 + lane]; };
    bf16x8 next_h[TS][NB <= 2 ? NB : 1], next_l[TS][NB <= 2 ? NB : 1];
    uint2 next_n[TS];
    auto preload = [&](int g, int tp) {
#pragma unroll
        for (int q = 0; q < TS; ++q) {
#pragma unroll
            for (int nb = 0; nb < (NB <= 2 ? NB : 1); ++nb) {
                next_l[q][nb] = operand(g, TS * tp + q, nb, 1);
                next_h[q][nb] = operand(g, TS * tp + q, nb, 0);
            }
            next_n[q] = nrm[g * 256 + (TS * tp + q) * 32 + col];
        }
    };
    // a word of every 128 bytes of a step's values: what is loaded one step later comes from the near cache
    uint32_t drawn[2] = {0u, 0u};
    auto draw_in = [&](int64_t chunk, int ml) {
        const rsrc_t rr = make_rsrc(x + chunk * 32 * d, (uint32_t)min<int64_t>(32, n - chunk * 32) * (uint32_t)d * 4u);
#pragma unroll
        for (int i = 0; i < 2; ++i) drawn[i] = __builtin_amdgcn_raw_buffer_load_b32(rr, col * d * 4 + half * 128 + i * 256, (m0 + ml) * ds * 4, 0);
    };
    take();
    if (AHEAD && chunk < chunks) fetch(chunk, ml);
    while (chunk < chunks) {
        if (!AHEAD) {
            asm volatile("" ::"v"(drawn[0]), "v"(drawn[1]));
            fetch(chunk, ml);
        }
        // ---- this step's operand
        bf16x8 bh[NB], bl[NB];
        float xx = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int j = ml * DSP + 16 * nb + 8 * half;
            const float4 u0 = *reinterpret_cast<const float4 *>(&mu[j]), u1 = *reinterpret_cast<const float4 *>(&mu[j + 4]);
            const f32x8 u = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
            const f32x8 v = raw[nb] - u;  // both are zero beyond the group
#pragma unroll
            for (int i = 0; i < 8; ++i) xx = fmaf(v[i], v[i], xx);
            split_bf16(v, bh[nb], bl[nb]);
        }
        const int64_t now = chunk;
        const int mlc = ml;
        if (++ml == mlend) take();
        if (NB <= 2) preload(mlc, 0);
        if (chunk < chunks) {
            if (AHEAD) fetch(chunk, ml);
            else draw_in(chunk, ml);
        }
        __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the matrix instructions
        // ---- all codewords, TS tiles at a time
        float tmax[8], rmax[16];
#pragma unroll
        for (int i = 0; i < 8; ++i) tmax[i] = -3.4e38f;
#pragma unroll
        for (int r = 0; r < 16; ++r) rmax[r] = -3.4e38f;
#pragma unroll
        for (int tp = 0; tp < 8 / TS; ++tp) {
            if (tp > 0 && K <= 32 * TS * tp) break;
            floatx16 acc[TS];
#pragma unroll
            for (int q = 0; q < TS; ++q) {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;
                constexpr int HB = NB >= 6 ? NB / 2 : NB;  // blocks whose small products come first (registers)
#pragma unroll
                for (int n0 = 0; n0 < NB; n0 += HB) {
                    bf16x8 ah[HB];
#pragma unroll
                    for (int i = 0; i < HB; ++i) {
                        ah[i] = NB <= 2 ? next_h[q][NB <= 2 ? i : 0] : operand(mlc, TS * tp + q, n0 + i, 0);
                        const bf16x8 al = NB <= 2 ? next_l[q][NB <= 2 ? i : 0] : operand(mlc, TS * tp + q, n0 + i, 1);
                        acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh[n0 + i], acc[q], 0, 0, 0);
                        acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[n0 + i], acc[q], 0, 0, 0);
                    }
#pragma unroll
                    for (int i = 0; i < HB; ++i) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[n0 + i], acc[q], 0, 0, 0);
                }
                // (the upper half's ones are zeros)
                const uint2 nn = NB <= 2 ? next_n[q] : nrm[mlc * 256 + (TS * tp + q) * 32 + col];
                acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, make_uint4(nn.x, nn.y, 0u, 0u)), ones, acc[q], 0, 0, 0);
            }
            if (NB <= 2 && tp < 3) preload(mlc, tp + 1);  // while the matrix cores work
#pragma unroll
            for (int r = 0; r < 16; ++r) rmax[r] = fmaxf(fmaxf(rmax[r], acc[0][r]), acc[1][r]);
#pragma unroll
            for (int q = 0; q < TS; ++q) {
                float t = acc[q][0];
#pragma unroll
                for (int r = 1; r < 15; r += 2) t = fmaxf(fmaxf(t, acc[q][r]), acc[q][r + 1]);
                tmax[TS * tp + q] = fmaxf(t, acc[q][15]);
                asm volatile("" : "+v"(tmax[TS * tp + q]));
            }
            // the maxima are taken here: put off until they are needed (as the compiler likes to), they keep the
            // accumulators of all tiles alive
#pragma unroll
            for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(rmax[r]));
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- decide.  Accumulator register r of lane l: codeword 32 tile + 8 (r / 4) + 4 (l / 32) + r % 4, vector l % 32
        {
            // the two halves of the wave hold different codewords of the same vectors: both halves' values in every lane
            auto halves = [](uint32_t a) { return __builtin_amdgcn_permlane32_swap(a, a, false, false); };
            float top = tmax[0];
#pragma unroll
            for (int i = 1; i < 8; ++i) top = fmaxf(top, tmax[i]);
            const auto tops = halves(__float_as_uint(top)), sums = halves(__float_as_uint(xx));
            top = fmaxf(__uint_as_float(tops[0]), __uint_as_float(tops[1]));
            const float norm = __uint_as_float(sums[0]) + __uint_as_float(sums[1]) + __uint_as_float(ccm[mlc]);
            const float E = eps * norm, th = top - E;
            // bits 16..23: tiles, 0..15: registers; the sign of maximum - threshold shifted in, one by one
            uint32_t mark = 0;
#pragma unroll
            for (int i = 7; i >= 0; --i) mark = __builtin_amdgcn_alignbit(mark, __float_as_uint(tmax[i] - th), 31);
#pragma unroll
            for (int r = 15; r >= 0; --r) mark = __builtin_amdgcn_alignbit(mark, __float_as_uint(rmax[r] - th), 31);
            mark = ~mark & 0x00FFFFFFu;
            // not finite, or so small that products vanish: every codeword goes through the rule
            if (!(E < inf) || norm < 1.0e-30f) mark = 0x00FFFFFFu;
            const int64_t v = now * 32 + col;
            const bool live = v < n;
            const auto marks = halves(mark);
            const uint32_t sel = marks[0] | marks[1];
            const bool hard = live && ((marks[0] && marks[1]) || __popc(sel) != 2);
            const int r = __ffs((int)(sel & 0xFFFFu)) - 1, tile = __ffs((int)(sel >> 16)) - 1;
            put(now, m0 + mlc, half == 0 && !hard, (uint32_t)(32 * tile + 8 * (r >> 2) + (marks[0] ? 0 : 4) + (r & 3)));
            const uint64_t hb = __ballot(hard);
            if (hb != 0ull) {
                const uint32_t lowm = (uint32_t)hb;  // both halves of the wave agree on which vectors are open
                const int nh = __popc(lowm);
                if (hcount + nh > 64) settle();
                const int slot = hcount + __popc(lowm & ((1u << col) - 1u));
                hcount += nh;
                if (hard && half == 0) {
                    hvec[slot] = ((uint64_t)v << 8) | (uint32_t)(m0 + mlc);
                    hbest[slot] = (uint64_t)0x7F7FFFFFu << 32;  // codeword 0 where no distance is below the largest float
                }
                uint32_t tm = hard ? mark >> 16 : 0u, rm = mark & 0xFFFFu;
                for (;;) {
                    const uint64_t pb = __ballot(tm != 0u);
                    if (pb == 0ull) break;
                    const int np = __popcll(pb);
                    if (pcount + np > ENC_PAIRS) evaluate();
                    if (tm != 0u) {
                        const int rr = __ffs((int)rm) - 1, tt = __ffs((int)tm) - 1;
                        const int at = pcount + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(pb >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pb, 0u));
                        pairs[at] = ((uint32_t)slot << 8) | (uint32_t)(32 * tt + 8 * (rr >> 2) + 4 * half + (rr & 3));
                        rm &= rm - 1u;
                        if (rm == 0u) {
                            tm &= tm - 1u;
                            rm = mark & 0xFFFFu;
                        }
                    }
                    pcount += np;
                }
            }
        }
    }
    settle();
}

// -0.5 ||c||^2 of every codeword (-3e38 beyond K) as cc2[M][256], and the largest ||c||^2 of every group as
// cc2[M * 256 + m]: what k_encode_wide starts its accumulators from.  grid (M), block 256.
__global__ __launch_bounds__(256) void k_encode_norms(const float *__restrict__ cb, int ds, int K, int M, float *__restrict__ cc2)
{
    __shared__ float s_mx[4];
    const int m = blockIdx.x, t = threadIdx.x;
    const float *c = cb + ((int64_t)m * K + t) * ds;
    float cc = 0.f;
    if (t < K)
        for (int j = 0; j < ds; ++j) cc = fmaf(c[j], c[j], cc);
    cc2[m * 256 + t] = t < K ? -0.5f * cc : -3.0e38f;
    float mx = t < K ? cc : 0.f;
#pragma unroll
    for (int dlt = 32; dlt > 0; dlt >>= 1) mx = fmaxf(mx, __shfl_xor(mx, dlt));
    if ((t & 63) == 0) s_mx[t >> 6] = mx;
    __syncthreads();
    if (t == 0) cc2[M * 256 + m] = fmaxf(fmaxf(s_mx[0], s_mx[1]), fmaxf(s_mx[2], s_mx[3]));
}

// ------------------------------------------------------------------------------------------------
// The matrix-core assignment for wide groups (more than 128 dimensions per group, aligned rows): both operands go
//     through LDS 32 dimensions at a time, fetched with coalesced 16-byte loads (eight threads per row) into registers
//     while the previous stage is multiplied, as in k_ivf_coarse_tc; k_encode_mfma's per-lane loads of 16 bytes from
//     64 different rows keep the matrix cores waiting for the cache's tag look-ups.  A workgroup owns 128 vectors
//     and the group's 256 codewords: wave (wk, wv) multiplies codewords 128 wk .. by vectors 64 wv .. (A = codewords,
//     4 x 2 accumulator blocks that start at -||c||^2 / 2), keeps the largest value, its index and the second largest per
//     vector (four instructions a value), the two waves of a vector set merge through LDS, and near-ties go through the
//     float32 rule.
//     The codes are k_encode's, bit for bit.
//     cc2: from k_encode_norms.  grid (ceil(n / 128), M), block 256; ds and d multiples of 4, K <= 256.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void k_encode_wide(const float *__restrict__ x, int64_t n, int d, int ds, int K, int M,
                                                        const float *__restrict__ cb, const float *__restrict__ cc2, uint8_t *__restrict__ codes)
{
    constexpr int RS = 36;  // floats per LDS row: 16 lanes reading one column of 16 rows hit 16 different bank quartets
    __shared__ __attribute__((aligned(16))) float tile[384 * RS];  // rows 0..127: vectors, 128..383: codewords
    __shared__ __align__(16) float s_cc2[256];
    __shared__ float s_v1[128], s_v2[128];
    __shared__ int s_k1[128];
    typedef float vf4 __attribute__((ext_vector_type(4)));
    const int t = threadIdx.x, lane = t & 63, w = uniform(t >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int wk = w & 1, wv = w >> 1;
    const int m = blockIdx.y;
    const int64_t v0 = (int64_t)blockIdx.x * 128;
    const float *cbm = cb + (int64_t)m * K * ds;
    const float *xw = x + v0 * d + (int64_t)m * ds;
    const int vrows = (int)min<int64_t>(128, n - v0);
    s_cc2[t] = cc2[m * 256 + t];
    // float4 number t + 256 i of a stage, i = 0..11, is piece t & 7 of row (t >> 3) + 32 i; rows beyond the data or
    // the codebook read the last one (their results are not used: -3e38 in cc2, no code written)
    const int r0 = t >> 3, c4 = t & 7;
    uint32_t off[12];
#pragma unroll
    for (int i = 0; i < 4; ++i) off[i] = (uint32_t)(min(r0 + 32 * i, vrows - 1) * d + 4 * c4);
#pragma unroll
    for (int i = 4; i < 12; ++i) off[i] = (uint32_t)(min(r0 + 32 * (i - 4), K - 1) * ds + 4 * c4);
    const int dst0 = r0 * RS + 4 * c4;
    vf4 st[12];
    auto fetch = [&](int j0) {
        const bool in = j0 + 4 * c4 + 4 <= ds;  // the group's last stage may be shorter: zeros beyond it
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            vf4 v = 0.f;
            if (in) v = *reinterpret_cast<const vf4 *>((i < 4 ? xw : cbm) + off[i] + j0);
            st[i] = v;
        }
    };
    fetch(0);
    __syncthreads();  // s_cc2
    floatx16 acc[4][2];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 c = *reinterpret_cast<const float4 *>(&s_cc2[wk * 128 + rb * 32 + 8 * g + 4 * half]);
#pragma unroll
            for (int cbk = 0; cbk < 2; ++cbk) {
                acc[rb][cbk][4 * g + 0] = c.x;
                acc[rb][cbk][4 * g + 1] = c.y;
                acc[rb][cbk][4 * g + 2] = c.z;
                acc[rb][cbk][4 * g + 3] = c.w;
            }
        }
    const int arow = 128 + wk * 128, brow = wv * 64;  // first LDS row of this wave's codewords and vectors
    float xx[2] = {0.f, 0.f};
    for (int j0 = 0; j0 < ds; j0 += 32) {
        __syncthreads();  // the previous stage has been read
#pragma unroll
        for (int i = 0; i < 12; ++i) *reinterpret_cast<vf4 *>(tile + dst0 + 32 * i * RS) = st[i];
        __syncthreads();
        fetch(min(j0 + 32, ((ds - 1) >> 5) << 5));  // after the last stage: the last again (not used)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the stage's matrix instructions
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            const int j = 16 * blk + 8 * half;
            float a[4][8], b[2][8];
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                const float *p = tile + (arow + rb * 32 + col) * RS + j;
                const float4 lo = *reinterpret_cast<const float4 *>(p), hi = *reinterpret_cast<const float4 *>(p + 4);
                a[rb][0] = lo.x; a[rb][1] = lo.y; a[rb][2] = lo.z; a[rb][3] = lo.w;
                a[rb][4] = hi.x; a[rb][5] = hi.y; a[rb][6] = hi.z; a[rb][7] = hi.w;
            }
#pragma unroll
            for (int cbk = 0; cbk < 2; ++cbk) {
                const float *p = tile + (brow + cbk * 32 + col) * RS + j;
                const float4 lo = *reinterpret_cast<const float4 *>(p), hi = *reinterpret_cast<const float4 *>(p + 4);
                b[cbk][0] = lo.x; b[cbk][1] = lo.y; b[cbk][2] = lo.z; b[cbk][3] = lo.w;
                b[cbk][4] = hi.x; b[cbk][5] = hi.y; b[cbk][6] = hi.z; b[cbk][7] = hi.w;
#pragma unroll
                for (int i = 0; i < 8; ++i) xx[cbk] = fmaf(b[cbk][i], b[cbk][i], xx[cbk]);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                    for (int cbk = 0; cbk < 2; ++cbk)
                        acc[rb][cbk] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[rb][i], b[cbk][i], acc[rb][cbk], 0, 0, 0);
        }
    }
    // accumulator register r of block rb, lane l: codeword 128 wk + 32 rb + 8 (r / 4) + 4 (l / 32) + r % 4, vector
    // 64 wv + 32 cbk + l % 32.  Largest and second largest value and the first index of the largest, per vector.
    const float inf = __uint_as_float(0x7F800000u);
    float v1[2], v2[2];
    int k1[2];
#pragma unroll
    for (int cbk = 0; cbk < 2; ++cbk) {
        float a1 = -3.0e38f, a2 = -3.0e38f;
        int kk = 0;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float val = acc[rb][cbk][r];
                kk = val > a1 ? rb * 32 + 8 * (r / 4) + (r % 4) : kk;
                a2 = __builtin_amdgcn_fmed3f(val, a1, a2);
                a1 = __builtin_amdgcn_fmed3f(val, a1, inf);
            }
        kk += wk * 128 + 4 * half;
        // the two halves of the wave saw different codewords of the same vectors
        const float o1 = __shfl_xor(a1, 32), o2 = __shfl_xor(a2, 32);
        const int ok = __shfl_xor(kk, 32);
        xx[cbk] += __shfl_xor(xx[cbk], 32);
        const float lo = fminf(a1, o1);
        if (o1 > a1 || (o1 == a1 && ok < kk)) kk = ok;
        v1[cbk] = fmaxf(a1, o1);
        v2[cbk] = fmaxf(lo, fmaxf(a2, o2));
        k1[cbk] = kk;
    }
    // the wave with the upper 128 codewords hands its result to the one with the lower 128
    if (wk == 1 && half == 0) {
#pragma unroll
        for (int cbk = 0; cbk < 2; ++cbk) {
            const int vi = wv * 64 + cbk * 32 + col;
            s_v1[vi] = v1[cbk];
            s_v2[vi] = v2[cbk];
            s_k1[vi] = k1[cbk];
        }
    }
    __syncthreads();
    if (wk == 1) return;
    const float ccmax = cc2[M * 256 + m];
    const float eps = 8.f * (float)(ds + 2) * 5.9604645e-8f;
#pragma unroll
    for (int cbk = 0; cbk < 2; ++cbk) {
        const int vi = wv * 64 + cbk * 32 + col;
        const float o1 = s_v1[vi], o2 = s_v2[vi];
        const int ok = s_k1[vi];
        const float lo = fminf(v1[cbk], o1);
        int kk = k1[cbk];
        if (o1 > v1[cbk] || (o1 == v1[cbk] && ok < kk)) kk = ok;
        const float b1 = fmaxf(v1[cbk], o1), b2 = fmaxf(lo, fmaxf(v2[cbk], o2));
        const int64_t v = v0 + vi;
        const bool live = v < n;
        const float E = eps * (xx[cbk] + ccmax);
        // (values so small that products are subnormal: the matrix instruction flushes them, E does not cover that)
        const bool hard = live && (!(b1 - b2 > E) || xx[cbk] + ccmax < 1.0e-30f);
        if (half == 0 && live && !hard) codes[v * M + m] = (uint8_t)kk;
        // near-ties: the float32 rule itself for every codeword, the wave's lanes taking codewords lane, lane + 64, ...
        uint64_t todo = __ballot(hard && half == 0);
        while (todo != 0ull) {
            const int src = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const int64_t vh = v0 + wv * 64 + cbk * 32 + src;
            const int best = encode_rule_wave(x + vh * d + (int64_t)m * ds, cbm, ds, K, lane, true);
            if (lane == 0) codes[vh * M + m] = (uint8_t)best;
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Consumers of a finished distance.  One distance belongs to (item, query lane).
// ------------------------------------------------------------------------------------------------
enum { OUT_ALLPAIRS = 0, OUT_SAMPLE = 1, OUT_FILTER = 2 };

struct OutArgs {
    // OUT_ALLPAIRS
    float *dist;        // [Q][N], rows q0.. of this batch
    int64_t N;          // row length
    int64_t nq;         // live queries of this batch (rows beyond are not written)
    // OUT_SAMPLE: the sample is cut into groups of `gsize` consecutive entries; only the minimum of
    // every group is kept
    float *gmin;        // [tiles*64][gstride]: a query's minima side by side, as k_tau reads them
    int64_t ngroups;
    int64_t gstride;    // ngroups rounded up to a multiple of 64
    int gsize;
    uint32_t *done;     // per block of 128 queries: not zero where k_mm16 has filtered it (k_lds16 takes the others), then as many
                        // words where k_tau says whose error bound is too large, then the number of the former; cleared by the
                        // sample pass of k_lds; or nullptr
    int blocks;         // the number of blocks
    int shares;         // workgroups per unit of the launch as the host cut it
    bool fixed;         // ... that many always (option lds_blocks)
    int wps;            // k_lds: waves that share a stretch of the sample (a power of two, at most 16)
    // OUT_FILTER
    const float *tau;   // [tiles*64]
    uint32_t *cnt;      // [tiles*64]
    uint64_t *cand;     // [tiles*64][C]
    uint32_t C;
    // Leaf payload (paper, Experiments: extra information stored on the leaf node): a term added to the finished sum
    // of an item, after the table entries.  term is indexed by the item's number in the array the kernel walks
    // (distinct entries, or input positions); where the kernel walks a stream that stands for other items (the
    // bound's sample stored side by side) term_map gives the item number of stream position i.  nullptr: none.
    const float *term;
    const uint32_t *term_map;
};

__device__ __forceinline__ void emit_filter(const OutArgs &o, int tile, int col, float tauv, float d, uint32_t item)
{
    if (d <= tauv) {
        const int64_t ql = (int64_t)tile * QT + col;
        const uint32_t pos = atomicAdd(&o.cnt[ql], 1u);
        if (pos < o.C) o.cand[ql * o.C + pos] = ((uint64_t)__float_as_uint(d) << 32) | item;
    }
}

// ------------------------------------------------------------------------------------------------
// B0  flat ADC: every encoding costs M lookups.  All M slices in LDS, lane = g*Qs + q.
//     items: ALLPAIRS -> n in [0,N) (input order); SAMPLE -> sample_pos[i]; FILTER -> n in [0,N).
//     grid (blocks, G, tiles).
// ------------------------------------------------------------------------------------------------
template <int G>
__device__ __forceinline__ float flat_one(const float *lds, const uint8_t *__restrict__ c, int M, int K, int qq)
{
    constexpr int Qs = WAVE / G;
    float acc = 0.f;
    if ((M & 3) == 0) {
        const uint32_t *c4 = reinterpret_cast<const uint32_t *>(c);
        for (int i = 0; i < (M >> 2); ++i) {
            const uint32_t dw = c4[i];
#pragma unroll
            for (int b = 0; b < 4; ++b) acc += lds[((i * 4 + b) * K + ((dw >> (8 * b)) & 255)) * Qs + qq];
        }
    } else {
        for (int m = 0; m < M; ++m) acc += lds[(m * K + c[m]) * Qs + qq];
    }
    return acc;
}

template <int G, int MODE>
__global__ void k_flat(const uint8_t *__restrict__ codes, int64_t nitems, const uint32_t *__restrict__ sample,
                       const float *__restrict__ lutT, int M, int K, int per_block, OutArgs o)
{
    constexpr int Qs = WAVE / G;
    extern __shared__ float lds[];
    const int tile = blockIdx.z, sub = blockIdx.y;
    stage_slices<G>(lds, lutT, tile, sub, M, K, 0, M);
    const int lane = threadIdx.x & 63;
    const int lg = lane / Qs, qq = lane % Qs;
    const int w = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int col = sub * Qs + qq;
    if (MODE == OUT_SAMPLE) {
        // every (wave, lane group) owns whole sample groups
        for (int64_t g = ((int64_t)blockIdx.x * nw + w) * G + lg; g < o.ngroups; g += (int64_t)gridDim.x * nw * G) {
            const int64_t lo = g * o.gsize, hi = min(nitems, lo + o.gsize);
            float best = __uint_as_float(0x7F800000u);
            for (int64_t j = lo; j < hi; ++j)
                best = fminf(best, flat_one<G>(lds, codes + (int64_t)sample[j] * M, M, K, qq) + (o.term ? o.term[sample[j]] : 0.f));
            o.gmin[((int64_t)tile * QT + col) * o.gstride + g] = best;
        }
        return;
    }
    const int64_t blo = (int64_t)blockIdx.x * per_block;
    const int64_t bhi = min(nitems, blo + per_block);
    float tauv = 0.f;
    if (MODE == OUT_FILTER) tauv = o.tau[(int64_t)tile * QT + col];
    for (int64_t j = blo + (int64_t)w * G + lg; j < bhi; j += (int64_t)nw * G) {
        const float acc = flat_one<G>(lds, codes + j * M, M, K, qq) + (o.term ? o.term[j] : 0.f);
        if (MODE == OUT_ALLPAIRS) {
            const int64_t ql = (int64_t)tile * QT + col;
            if (ql < o.nq) o.dist[ql * o.N + j] = acc;
        } else {
            emit_filter(o, tile, col, tauv, acc, (uint32_t)j);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Search and all-pairs output with every table slice in LDS (flat ADC, and the trees walked by the waves).
//     All M = 4*M4 slices of a sub-tile of Qs = 64/G queries are staged in LDS (as lines, see stage_lines);
//     a lane owns V = 4 adjacent queries of one item, so one address and one 16-byte LDS read serve four
//     distances: Qs/4 lanes per item (a lane group), IPS = 4G items per wave step (measured on cfg2:
//     V = 1, 2, 4, 8 -> 12.2, 4.2, 3.5, 4.8 ms).  Nothing but the item records is read from HBM.
//     The sum of an item: see lds_item_sum (chunks in pairs inside the groups of a line, groups and trees in
//     order).
//
//     OUT_FILTER: a workgroup takes per_block consecutive items and cuts them into one run per wave; the
//     wave's lane groups take the run's items in turn.  With CTX the items are the sorted distinct
//     encodings and every lane group carries a Distance Context (paper, "Distance Computation with
//     Hierarchical Memory Structure") over the items it sees, reduced to the first two levels of tree 0: as
//     long as no lane group of the wave leaves the 2-chunk prefix of its previous item, the sum over those
//     levels is kept and only the deeper chunks are looked up; otherwise the whole wave recomputes it
//     (which changes nothing for the lane groups that did not need to).  Deeper levels are not shared: the
//     lane groups of a wave diverge there almost every step, and a lookup costs the same whether or not
//     every group needs it.
//     Candidates at or below the bound go to a ring of the wave in LDS (slot = rank among the passing
//     lanes) and are appended to the queries' lists by the whole wave when the ring is nearly full: one
//     global reservation per query, then LDS atomics hand out the slots.
//     OUT_SAMPLE: items map[i] (or i itself without a map: the sample's records stored side by side); a wave
//     walks a stretch of the sample, every lane group's share of it is one sample group, whose minimum it keeps.
//     OUT_ALLPAIRS: items are input positions (rec = the codes in input order, no context); a lane group takes
//     U consecutive positions, so dist[q][n] is written in pieces of U floats per lane, U * IPS adjacent floats
//     of a row per store instruction.
//     rec [n][M4] dwords: the codes of an item, chunk 0 in the lowest byte.
//     grid (blocks, G, tiles), block 1024, dynamic LDS lds_table_bytes + lds_aux_bytes, no static LDS;
//     per_block < 2^26.
// ------------------------------------------------------------------------------------------------
constexpr int LDS_V = 4;  // queries per lane (one 16-byte LDS read per lookup)
typedef float vecq __attribute__((ext_vector_type(LDS_V)));

// Sum of one item.  The chunks are taken in groups of CPL = 4 or 8 (the chunks of one LDS line), a group as a
// balanced tree, (x0 + x1) + (x2 + x3) or ((x0 + x1) + (x2 + x3)) + ((x4 + x5) + (x6 + x7)), where x0 .. are the
// group's entries in the order the lane read them.  That order differs from lane group to lane group (see
// k_lds), but only by exchanging the two halves of subtrees of that tree (read order = t XOR j), and float
// addition is commutative: every lane forms exactly the tree over c0 .. c(CPL-1), bit for bit.  With CPL = 4 a
// tree's sum is the sum of its groups in order (a tree of fewer than four chunks lives inside one group) and
// the trees are added in order; with CPL = 8 the groups are added in order.
// CTX: `top` is the first pair of group 0, c0 + c1; with fast it is reused instead of read.
template <int M4, int T, int CPL, bool CTX, class Look>
__device__ __forceinline__ vecq lds_item_sum(Look look, bool fast, vecq &top)
{
    constexpr int NG = 4 * M4 / CPL;
    constexpr int D = 4 * M4 / T;
    constexpr int GPT = CPL == 8 ? NG : (D >= 4 ? D / 4 : 1);  // groups per tree
    vecq P[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        vecq a;
        if (CTX && g == 0) {
            if (fast) {
                a = top;
            } else {
                a = look(g, 0) + look(g, 1);
                top = a;
            }
        } else {
            a = look(g, 0) + look(g, 1);
        }
        P[g] = a + (look(g, 2) + look(g, 3));
        if (CPL == 8) P[g] = P[g] + ((look(g, 4) + look(g, 5)) + (look(g, 6) + look(g, 7)));
    }
    vecq d = 0.f;
#pragma unroll
    for (int t0 = 0; t0 < NG; t0 += GPT) {
        vecq s = P[t0];
#pragma unroll
        for (int i = 1; i < GPT; ++i) s += P[t0 + i];
        d = t0 == 0 ? s : d + s;
    }
    return d;
}

// The same sum on fixed-point entries (see k_lds, FX): integer addition is associative, so the order in which a lane
// reads the chunks does not matter and three entries go into one add.  CTX: `top` is the sum of chunks 0 and 1.
typedef uint32_t vecu4 __attribute__((ext_vector_type(LDS_V)));
template <int M4, int CPL, bool CTX, class Look>
__device__ __forceinline__ vecu4 lds_item_sum_fx(Look look, bool fast, vecu4 &top)
{
    constexpr int NG = 4 * M4 / CPL;
    vecu4 d;
    if (CTX) {
        if (!fast) top = look(0, 0) + look(0, 1);
        d = top;
    } else {
        d = look(0, 0) + look(0, 1);
    }
#pragma unroll
    for (int t = 2; t < CPL; t += 2) d = d + look(0, t) + look(0, t + 1);
#pragma unroll
    for (int g = 1; g < NG; ++g)
#pragma unroll
        for (int t = 0; t < CPL; t += 2) d = d + look(g, t) + look(g, t + 1);
    return d;
}

// Fixed-point form of a table entry for the candidate filter of k_lds: entries are scaled so that the query's bound
// becomes FX_TOP and cut off at FX_CAP (an entry beyond twice the bound cannot belong to a candidate); M <= 16
// capped entries add up to less than 2^32.
constexpr float FX_TOP = 134217728.f;        // 2^27
constexpr uint32_t FX_CAP = (1u << 28) - 1u;
__device__ __forceinline__ float fx_scale(float tau) { return FX_TOP / fmaxf(tau, 8.0779e-28f /* 2^-90 */); }
__device__ __forceinline__ uint32_t fx_entry(float e, float scale, bool dead)
{
    const uint32_t v = (uint32_t)fminf(e * scale, (float)FX_CAP);  // truncates; the float cap rounds to 2^28
    return dead ? FX_CAP : min(v, FX_CAP);
}
// Largest sum the filter lets through.  An item whose float32 distance d (any order of additions) is at or below
// tau has a real sum of entries of at most d (1 + M 2^-24); every fixed-point entry is at most its real product with
// the scale times (1 + 2^-24).  (1 + 2^-19) covers both for M <= 16, and the + 2 the rounding of this product.
__device__ __forceinline__ uint32_t fx_bound(float tau, float scale)
{
    if (!(tau >= 0.f)) return 0u;  // a dead query column: every entry is FX_CAP there, nothing passes
    return (uint32_t)fminf(tau * scale * (1.f + 1.9073486e-6f), 4.0e9f) + 2u;
}

// chunks per LDS line of the LDS-resident kernels: a line is at least 256 bytes (all banks)
__host__ __device__ constexpr int lds_chunks_per_line(int G) { return G == 8 ? 8 : 4; }

// Stages all M slices of sub-tile g as lines: the rows of the CPL chunks of a group (same codeword number) side
// by side, [M/CPL][KP][CPL][Qs].  With rows of 64 (32) bytes and CPL = 4 (8) a line is 256 bytes = all LDS
// banks, so the row of chunk m always sits in the same bank quarter (eighth) m % CPL, whatever the codeword.
// KP >= K is the number of lines reserved per group.
// FX: the entries are stored in fixed point (fx_entry) with the scale of their query, tau = the bounds of the tile.
template <int G, bool FX = false>
__device__ __forceinline__ void stage_lines(float *lds, const float *__restrict__ lutT, int tile, int g, int M, int K, int KP,
                                            const float *__restrict__ tau = nullptr)
{
    // 16 bytes per load and store, eight loads in flight per thread before the first store: a workgroup of 1024
    // threads moves the 128 KB of a sub-tile in one trip
    constexpr int Qs = WAVE / G, CPL = lds_chunks_per_line(G), P4 = Qs / 4, UN = 8;
    const int total = M * K * P4;  // 16-byte pieces: row (m, k) has P4 of them
    const float *src = lutT + (int64_t)tile * M * K * QT + g * Qs;
    // a thread always handles the same piece p of a row (the block size and the trip are multiples of P4): the four
    // queries whose scales it needs
    float sc[4] = {0.f, 0.f, 0.f, 0.f};
    bool dead[4] = {false, false, false, false};
    if (FX) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float t = tau[(int64_t)tile * QT + g * Qs + ((int)threadIdx.x % P4) * 4 + v];
            dead[v] = !(t >= 0.f);
            sc[v] = fx_scale(t);
        }
    }
    auto put = [&](int idx, float4 v) {
        const int row = idx / P4, p = idx % P4;  // row = m * K + k
        const int m = K == 256 ? row >> 8 : row / K, k = row - m * K;
        if (FX) {
            v.x = __uint_as_float(fx_entry(v.x, sc[0], dead[0]));
            v.y = __uint_as_float(fx_entry(v.y, sc[1], dead[1]));
            v.z = __uint_as_float(fx_entry(v.z, sc[2], dead[2]));
            v.w = __uint_as_float(fx_entry(v.w, sc[3], dead[3]));
        }
        *reinterpret_cast<float4 *>(lds + (((m / CPL) * KP + k) * CPL + (m % CPL)) * Qs + p * 4) = v;
    };
    const int trip = (int)blockDim.x * UN;
    int base = 0;
    for (; base + trip <= total; base += trip) {  // whole trips: no bounds checks between the loads
        float4 v[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int idx = base + u * (int)blockDim.x + (int)threadIdx.x;
            v[u] = *reinterpret_cast<const float4 *>(src + (int64_t)(idx / P4) * QT + (idx % P4) * 4);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) put(base + u * (int)blockDim.x + (int)threadIdx.x, v[u]);
    }
    for (int idx = base + (int)threadIdx.x; idx < total; idx += (int)blockDim.x)
        put(idx, *reinterpret_cast<const float4 *>(src + (int64_t)(idx / P4) * QT + (idx % P4) * 4));
    __syncthreads();
}

// bytes of LDS k_lds needs: the table lines, and behind them the candidate ring and its counters in filter mode
constexpr int LDS_RING = 160;
__host__ __device__ inline int lds_lines_per_group(int G, int K) { return (G == 4 || G == 8) ? 256 : K; }
__host__ __device__ inline size_t lds_table_bytes(int G, int M, int K)
{
    const int CPL = lds_chunks_per_line(G);
    return (size_t)(M / CPL) * lds_lines_per_group(G, K) * (size_t)(CPL * (WAVE / G) * 4);
}
__host__ __device__ inline size_t lds_aux_bytes(bool filter) { return filter ? (size_t)16 * LDS_RING * 8 + 2 * 16 * 64 * 4 : 0; }
constexpr size_t LDS_SAMPLE_BYTES = 16 * 64 * 16;  // sample mode with shared stretches: a partial minimum per lane
// k_lds16: a ring entry is a lane's eight results (16 bytes) and a word that says whose they are
constexpr int LDS16_RING = 76;
__host__ __device__ inline size_t lds16_aux_bytes() { return (size_t)16 * LDS16_RING * 20 + 2 * 16 * 64 * 4 + 16; }

typedef __attribute__((address_space(3))) const vecq lds_vecq_t;

template <int G, int M4, int T, int MODE, bool CTX, bool FX = false, bool TERM = false>
__global__ __launch_bounds__(1024) void k_lds(const uint32_t *__restrict__ rec, int64_t nitems,
                                              const uint32_t *__restrict__ map, const float *__restrict__ lutT, int K,
                                              int per_block, OutArgs o)
{
    constexpr int Qs = WAVE / G, V = LDS_V, LPI = Qs / V, IPS = WAVE / LPI, M = 4 * M4;
    constexpr int S = CTX ? 2 : 0;  // chunks kept in the context: the first pair
    constexpr int U = M4 >= 4 ? 2 : 4;  // steps unrolled
    constexpr int RING = LDS_RING;
    constexpr bool FILTER = MODE == OUT_FILTER;
    // With rows of 64 bytes a line is 256 bytes, and with 256 lines per group the byte address of an entry is
    // (group << 16) | (code << 8) | (chunk << 6) | (lane's piece << 4): one v_perm_b32 drops the code byte of the
    // record into byte 1 of a per-lane constant, instead of a bit-field extract and a shift-add.  That needs the
    // tables at LDS address 0: this kernel has no static LDS, ring and counters live behind the tables.
    constexpr int CPL = lds_chunks_per_line(G), NG = M / CPL;
    constexpr bool PERM = CPL * Qs * 4 == 256;
    extern __shared__ float lds[];
    const int KP = PERM ? 256 : K;
    const uint32_t rowB = Qs * 4, lineB = CPL * rowB;
    char *aux = reinterpret_cast<char *>(lds) + (size_t)NG * KP * lineB;
    uint64_t(*ring)[RING] = reinterpret_cast<uint64_t(*)[RING]>(aux);
    uint32_t(*wcount)[64] = reinterpret_cast<uint32_t(*)[64]>(aux + 16 * RING * 8);
    uint32_t(*wpos)[64] = reinterpret_cast<uint32_t(*)[64]>(aux + 16 * RING * 8 + 16 * 64 * 4);
    const int tile = blockIdx.z, sub = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int w = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
    static_assert(!FX || MODE == OUT_FILTER, "the fixed-point form is a candidate filter");
    static_assert(!TERM || (MODE == OUT_FILTER && !FX), "TERM selects the filter pass with a leaf payload; the other modes test o.term");
    if (MODE == OUT_SAMPLE && o.done && blockIdx.x + blockIdx.y + blockIdx.z == 0)
        for (int i = threadIdx.x; i < 2 * o.blocks + 1; i += blockDim.x) o.done[i] = 0u;
    // a sub-tile past the last query: nothing to write
    if ((MODE == OUT_ALLPAIRS || MODE == OUT_SAMPLE) && (int64_t)tile * QT + sub * Qs >= o.nq) return;
    if (FILTER) wcount[w][lane] = 0u;
    stage_lines<G, FX>(lds, lutT, tile, sub, M, K, KP, FX ? o.tau : nullptr);
    const int lg = lane / LPI, lq = lane % LPI;
    const int col = sub * Qs + lq * V;  // first of this lane's queries inside the tile
    // Which chunk of a group this lane reads t-th: t ^ j with j = the lane group's number mod CPL.  The CPL lane
    // groups that share a pass of the LDS pipe (16 lanes x 16 bytes) then read CPL different chunks at any time,
    // i.e. different bank quarters (eighths): no bank conflicts, whatever the codes.  Group 0 of a walk with
    // context only swaps inside its pairs (and, with CPL = 8, rotates chunks 4 .. 7 among themselves), so that the
    // first two reads are chunks 0 and 1 in every lane and can be skipped together.
    const int jr = lg & (CPL - 1);
    const uint32_t base = (uint32_t)(uintptr_t)lds;  // LDS address of the tables (0 when PERM)
    uint32_t sh[2][CPL];   // PERM: selector of v_perm_b32; else shift of the code byte.  [0]: group 0, [1]: the others
    uint32_t pb[NG][CPL];  // LDS address of line 0 of that chunk for this lane
#pragma unroll
    for (int t = 0; t < CPL; ++t) {
        int c0 = t ^ jr;
        if (CTX) c0 = t < 4 ? (t ^ (jr & 1)) : 4 + ((t - 4) ^ (jr & 3));
        const int c1 = t ^ jr;
        sh[0][t] = PERM ? (0x03020000u | ((4u + (uint32_t)(c0 & 3)) << 8)) : 8u * (uint32_t)(c0 & 3);
        sh[1][t] = PERM ? (0x03020000u | ((4u + (uint32_t)(c1 & 3)) << 8)) : 8u * (uint32_t)(c1 & 3);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int c = g == 0 ? c0 : c1;
            pb[g][t] = base + (uint32_t)(lq * (V * 4)) + (uint32_t)g * (uint32_t)KP * lineB + (uint32_t)c * rowB;
        }
    }
    // CPL = 8: the two record dwords of a group; a lane whose rotation exchanges the halves reads them crosswise
    const bool cross = CPL == 8 && (jr & 4) != 0;
    typedef __attribute__((address_space(3))) const vecu4 lds_vecu4_t;
    // LDS address of the t-th entry a lane reads of group g of an item
    auto addr_of = [&](const uint32_t dw[M4], int g, int t) -> uint32_t {
        uint32_t src;
        if (CPL == 4) {
            src = dw[g];
        } else {
            const bool second = (CTX && g == 0) ? t >= 4 : ((t >= 4) != cross);
            src = second ? dw[2 * g + 1] : dw[2 * g];
        }
        if (PERM) return __builtin_amdgcn_perm(src, pb[g][t], sh[g == 0 ? 0 : 1][t]);
        return pb[g][t] + __builtin_amdgcn_ubfe(src, sh[g == 0 ? 0 : 1][t], 8) * lineB;
    };
    auto sum_of_fx = [&](const uint32_t dw[M4], bool fast, vecu4 &top) -> vecu4 {
        auto look = [&](int g, int t) -> vecu4 { return *reinterpret_cast<lds_vecu4_t *>(addr_of(dw, g, t)); };
        return lds_item_sum_fx<M4, CPL, CTX>(look, CTX && fast, top);
    };
    auto sum_of = [&](const uint32_t dw[M4], bool fast, vecq &top) -> vecq {
        auto look = [&](int g, int t) -> vecq {
            uint32_t src;
            if (CPL == 4) {
                src = dw[g];
            } else {
                const bool second = (CTX && g == 0) ? t >= 4 : ((t >= 4) != cross);
                src = second ? dw[2 * g + 1] : dw[2 * g];
            }
            uint32_t addr;
            if (PERM) {
                // bytes 0, 2, 3 from pb (byte 1 of pb is zero), byte 1 = the code: selector bytes 0..3 pick from
                // the second operand, 4..7 from the first
                addr = __builtin_amdgcn_perm(src, pb[g][t], sh[g == 0 ? 0 : 1][t]);
            } else {
                addr = pb[g][t] + __builtin_amdgcn_ubfe(src, sh[g == 0 ? 0 : 1][t], 8) * lineB;
            }
            return *reinterpret_cast<lds_vecq_t *>(addr);
        };
        return lds_item_sum<M4, T, CPL, CTX>(look, CTX && fast, top);
    };

    if (MODE == OUT_SAMPLE) {
        // The sample is cut into one stretch per IPS sample groups; a wave walks a stretch, its lane groups
        // taking the items in turn (coalesced record loads), and every lane group's share is one sample group.
        // (Any partition of the sample into ngroups disjoint sets serves the bound; the sample is in random
        // order.)  Where a batch has too few sub-tiles to fill the chip with a wave per stretch, wps waves of the
        // workgroup share one: each walks every wps-th block of steps, and their minima meet in LDS (one query
        // against a million vectors: 55 us with the 64 stretches walked by two workgroups, 7 us by 64).
        const int64_t nwr = (o.ngroups + IPS - 1) / IPS;
        const int64_t per = ((nitems + nwr - 1) / nwr + IPS - 1) / IPS * IPS;  // items per stretch
        const int wps = o.wps, sw = w & (wps - 1);
        auto walk = [&](int64_t wr) -> vecq {
            const int64_t lo = wr * per, hi = min(nitems, lo + per);
            vecq best = __uint_as_float(0x7F800000u);
            for (int64_t j0 = lo + (int64_t)sw * (IPS * U); j0 < hi; j0 += (int64_t)wps * (IPS * U)) {
                uint32_t dw[U][M4];
                bool live[U];
                float tm[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t idx = j0 + u * IPS + lg;
                    live[u] = idx < hi;
                    const int64_t ic = min(idx, nitems - 1);
                    const int64_t e = map ? (int64_t)map[ic] : ic;
#pragma unroll
                    for (int i = 0; i < M4; ++i) dw[u][i] = rec[e * M4 + i];
                    tm[u] = o.term ? o.term[o.term_map ? (int64_t)o.term_map[ic] : e] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    vecq top = 0.f;
                    const vecq d = sum_of(dw[u], false, top) + tm[u];
                    if (live[u]) {
#pragma unroll
                        for (int v = 0; v < V; ++v) best[v] = fminf(best[v], d[v]);
                    }
                }
            }
            return best;
        };
        auto keep = [&](int64_t wr, const vecq &best) {
            const int64_t g = wr * IPS + lg;
            if (g < o.ngroups) {
                float *dst = o.gmin + ((int64_t)tile * QT + col) * o.gstride + g;
#pragma unroll
                for (int v = 0; v < V; ++v) dst[v * o.gstride] = best[v];
            }
        };
        if (wps == 1) {
            for (int64_t wr = (int64_t)blockIdx.x * nw + w; wr < nwr; wr += (int64_t)gridDim.x * nw) keep(wr, walk(wr));
        } else {
            // one stretch per wps waves, no loop: the launch has waves for all of them
            const int64_t wr = ((int64_t)blockIdx.x * nw + w) / wps;
            vecq *part = reinterpret_cast<vecq *>(aux);  // [16 waves][64 lanes]
            vecq best = __uint_as_float(0x7F800000u);
            if (wr < nwr) best = walk(wr);
            part[w * WAVE + lane] = best;
            __syncthreads();
            if (sw == 0 && wr < nwr) {
                for (int i = 1; i < wps; ++i) {
                    const vecq b = part[(w + i) * WAVE + lane];
#pragma unroll
                    for (int v = 0; v < V; ++v) best[v] = fminf(best[v], b[v]);
                }
                keep(wr, best);
            }
        }
        return;
    }

    if (MODE == OUT_ALLPAIRS) {
        // items are the N input positions, U * IPS consecutive ones per wave and round; lane group g takes the U
        // consecutive items U g .. U g + U - 1, so that a lane ends up with U adjacent floats of each of its rows
        // and writes them as one piece: a store instruction of the wave covers U * IPS adjacent floats (256
        // bytes at U = 4) of four rows.  (The workgroups of a sub-tile take turns along the rows, so that what
        // is written at any time is close.)  Rows that are not 16-byte aligned get single floats.
        typedef float vecu __attribute__((ext_vector_type(U)));
        const int64_t bhi = nitems;
        const bool wide = (o.N % U) == 0 && (reinterpret_cast<uintptr_t>(o.dist) % (U * 4)) == 0;
        for (int64_t j0 = ((int64_t)blockIdx.x * nw + w) * (IPS * U); j0 < bhi; j0 += (int64_t)gridDim.x * nw * (IPS * U)) {
            uint32_t dw[U][M4];
            float tm[U];
            const int64_t jf = j0 + U * lg;  // this lane group's first item
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t j = min(jf + u, nitems - 1);
#pragma unroll
                for (int k2 = 0; k2 < M4; ++k2) dw[u][k2] = rec[j * M4 + k2];
                tm[u] = o.term ? o.term[j] : 0.f;
            }
            vecq d[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                vecq top = 0.f;
                d[u] = sum_of(dw[u], false, top) + tm[u];
            }
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const int64_t ql = (int64_t)tile * QT + col + v;
                if (ql >= o.nq) continue;
                float *row = o.dist + ql * o.N;
                if (wide && jf + U <= bhi) {  // written once, never read here
                    vecu x;
#pragma unroll
                    for (int u = 0; u < U; ++u) x[u] = d[u][v];
                    __builtin_nontemporal_store(x, reinterpret_cast<vecu *>(row + jf));
                } else {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (jf + u < bhi) __builtin_nontemporal_store(d[u][v], row + jf + u);
                }
            }
        }
        return;
    }

    const int64_t blo = (int64_t)blockIdx.x * per_block;
    const int64_t bhi = min(nitems, blo + per_block);
    // the bound of each of this lane's queries: as a float, or (FX) as the largest fixed-point sum that may pass
    float tau[V];
    uint32_t itau[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        tau[v] = o.tau[(int64_t)tile * QT + col + v];
        itau[v] = FX ? fx_bound(tau[v], fx_scale(tau[v])) : 0u;
    }
    int held = 0;
    // The ring holds (value bits << 32 | query of the tile << 26 | item relative to blo), wcount the entries per
    // query.  When the ring is nearly full the whole wave appends it to the queries' lists: one global reservation
    // per query (64 lanes, 64 queries), then LDS atomics hand out the slots.  (One global atomic per entry, all
    // workgroups of a sub-tile hitting the same 16 counters, cost 0.7 ms on the benchmark's 2.3 ms.)
    auto flush = [&]() {
        const uint32_t c = wcount[w][lane];
        wpos[w][lane] = c ? atomicAdd(&o.cnt[(int64_t)tile * QT + lane], c) : 0u;
        wcount[w][lane] = 0u;
        __builtin_amdgcn_wave_barrier();
        for (int i = lane; i < held; i += 64) {
            const uint64_t e = ring[w][i];
            const int owner = (int)((e >> 26) & 63u);
            const uint32_t pos = atomicAdd(&wpos[w][owner], 1u);
            const int64_t q = (int64_t)tile * QT + owner;
            if (pos < o.C)
                o.cand[q * o.C + pos] = (e & 0xFFFFFFFF00000000ull) | (uint32_t)(blo + (int64_t)(e & 0x3FFFFFFull));
        }
        __builtin_amdgcn_wave_barrier();
        held = 0;
    };
    auto emit = [&](bool pass, uint32_t bits, int c, uint32_t rel) {
        const uint64_t mask = __ballot(pass);
        if (mask != 0ull) {
            const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (pass) {
                ring[w][held + rank] = ((uint64_t)bits << 32) | ((uint32_t)c << 26) | rel;
                atomicAdd(&wcount[w][c], 1u);
            }
            held += __popcll(mask);
            if (held > RING - 64) flush();
        }
    };
    // A wave walks one run of consecutive items, its IPS lane groups taking the items in turn (lane group g:
    // items g, g + IPS, ...): a step reads IPS consecutive records, one coalesced load, and a CU follows 16
    // record streams.  (One run per lane group means 256 to 512 streams per CU; at 32 items per step they
    // overflow the 32 KB vector cache and every record load goes to L2: cfg4 72 -> 37 ms.)  The context of a lane
    // group then refers to the item IPS places back.  Records come through a buffer over the workgroup's
    // share, the step number in the scalar offset.
    constexpr int RF = IPS;  // lane groups per run
    if (blo >= bhi) return;
    const int nruns = nw * IPS / RF;
    const int RLr = (per_block + nruns - 1) / nruns;         // items per run
    const int RL = (RLr + RF - 1) / RF;                      // steps per run
    const int ph = lg % RF;
    const int64_t rlo = blo + (int64_t)((w * IPS + lg) / RF) * RLr;
    const int runlen = (int)max<int64_t>(0, min<int64_t>(bhi - rlo, RLr));
    const int len = runlen > ph ? (runlen - ph + RF - 1) / RF : 0;  // items of this lane group
    int minlen = len;
#pragma unroll
    for (int dlt = LPI; dlt < WAVE; dlt <<= 1) minlen = min(minlen, __shfl_xor(minlen, dlt));
    minlen = uniform(minlen);
    const rsrc_t rr = make_rsrc(rec + blo * M4, (uint32_t)((bhi - blo) * (M4 * 4)));
    const uint32_t first = (uint32_t)(rlo - blo) + (uint32_t)ph;   // this lane group's first item, relative to blo
    const uint32_t voff = len > 0 ? first * (M4 * 4) : 0u;
    uint32_t prev0 = 0u;
    vecq top = 0.f;
    vecu4 itop = 0u;
    // U steps from step i on; CHECK: some lane groups may be past the end of their run
    auto steps = [&](int i, auto check) {
        constexpr bool CHECK = decltype(check)::value;
        uint32_t dw[U][M4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t vo = voff;
            int so = (i + u) * (RF * M4 * 4);
            if (CHECK) {
                vo += (uint32_t)max(0, min(i + u, len - 1)) * (RF * M4 * 4);
                so = 0;
            }
#pragma unroll
            for (int k2 = 0; k2 < M4; ++k2) dw[u][k2] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rr, (int)vo + 4 * k2, so, 0);
        }
        if constexpr (FX && CTX && CPL == 4 && M4 == 2) {
            // The table reads of step u + 1 are issued before the entries of step u are added up and tested, so that
            // the LDS pipe, which bounds this kernel, always has reads of this wave queued (one workgroup of 16 waves
            // per CU cannot hide a read's latency by switching waves alone).  Only the six reads every step needs
            // are kept in flight (2 x 24 registers); the two of the context's chunks are read when a step renews it.
            bool fastv[U];  // which steps may keep the context (see below)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool live = !CHECK || i + u < len;
                const bool differs = live && ((dw[u][0] ^ prev0) & 0xFFFFu) != 0u;
                fastv[u] = __ballot(differs) == 0ull && i + u != 0;
                prev0 = dw[u][0];
            }
            vecu4 xr[2][M - 2];
            auto issue = [&](int u, vecu4 *x) {
#pragma unroll
                for (int t = 2; t < M; ++t) x[t - 2] = *reinterpret_cast<lds_vecu4_t *>(addr_of(dw[u], t / CPL, t % CPL));
            };
            issue(0, xr[0]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u + 1 < U) issue(u + 1, xr[(u + 1) & 1]);
                if (!fastv[u])
                    itop = *reinterpret_cast<lds_vecu4_t *>(addr_of(dw[u], 0, 0)) + *reinterpret_cast<lds_vecu4_t *>(addr_of(dw[u], 0, 1));
                const vecu4 *x = xr[u & 1];
                vecu4 d = itop + x[0] + x[1];
                d = d + x[2] + x[3];
                d = d + x[4] + x[5];
                const bool live = !CHECK || i + u < len;
                const uint32_t rel = first + (uint32_t)(i + u) * RF;
#pragma unroll
                for (int v = 0; v < V; ++v) emit(live && d[v] <= itau[v], d[v], col + v, rel);
            }
            return;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = !CHECK || i + u < len;
            bool fast = false;
            if (S > 0) {
                // a lane group may keep its context if its item has the S-chunk prefix of its previous one
                const uint32_t smask = S == 1 ? 0xFFu : 0xFFFFu;
                const bool differs = live && ((dw[u][0] ^ prev0) & smask) != 0u;
                fast = __ballot(differs) == 0ull && i + u != 0;
                prev0 = dw[u][0];
            }
            const uint32_t rel = first + (uint32_t)(i + u) * RF;
            if (FX) {
                const vecu4 d = sum_of_fx(dw[u], fast, itop);
#pragma unroll
                for (int v = 0; v < V; ++v) emit(live && d[v] <= itau[v], d[v], col + v, rel);
            } else {
                vecq d = sum_of(dw[u], fast, top);
                if (TERM) d += o.term[min(blo + (int64_t)rel, nitems - 1)];  // leaf payload: an instance of its own (a load per step)
#pragma unroll
                for (int v = 0; v < V; ++v) emit(live && d[v] <= tau[v], __float_as_uint(d[v]), col + v, rel);
            }
        }
    };
    int i = 0;
    for (; i + U <= minlen; i += U) steps(i, std::false_type{});
    for (; i < RL; i += U) steps(i, std::true_type{});
    flush();
}

// ------------------------------------------------------------------------------------------------
// Who works on what where a filter pass is divided between k_mm16 and k_lds16 on the device: workgroup `wg` of `wgs` finds
// its share of the items of its unit among the units that are left (block b has weight(b) of them).  The host sizes the launch
// for all units; a few that are left get more shares each, so that they still fill the compute units.  The shares are chosen by
// the rule of lds_blocks_for on the host (`given` > 0: that many), a candidate per lane.  (A launch cut for all of 79 blocks
// gave a single one 16 long workgroups: a whole round of the pass, 4 ms of 20.)  Every wave finds the same; the answer is uniform.
// (Where all units are left, or none, the kernels know it without.)
// ------------------------------------------------------------------------------------------------
constexpr int MM_Q = 128;  // queries per block of the divided pass
struct Share {
    int block, nth;     // the unit: the nth of its block
    int share, shares;
};
template <class F>
__device__ __forceinline__ bool find_share(uint32_t wg, uint32_t wgs, int blocks, int64_t nitems, int given, F weight, Share &s)
{
    const int lane = threadIdx.x & 63;
    uint32_t total = 0;
    for (int b0 = 0; b0 < blocks; b0 += 64) {
        uint32_t v = b0 + lane < blocks ? (uint32_t)weight(b0 + lane) : 0u;
#pragma unroll
        for (int dlt = 32; dlt >= 1; dlt >>= 1) v += (uint32_t)__shfl_xor((int)v, dlt);
        total += v;
    }
    total = (uint32_t)uniform((int)total);
    if (total == 0u) return false;
    uint32_t shares = (uint32_t)given;
    if (given == 0) {
        const uint32_t least = (uint32_t)(nitems >> 25) + 1u, most = max(least, (uint32_t)((nitems + 4095) / 4096));
        float cost = __uint_as_float(0x7F800000u);
        shares = least;  // (the launch has room for it)
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            const uint32_t n = least + i * 64u + (uint32_t)lane;
            if (n > least && (n > most || n > wgs / total || total * (n - 1u) >= 16u * 256u)) continue;
            const float c = (float)((total * n + 255u) / 256u) * (5000.f + (float)nitems / (float)n);
            if (c < cost) {
                cost = c;
                shares = n;
            }
        }
#pragma unroll
        for (int dlt = 32; dlt >= 1; dlt >>= 1) {
            const float oc = __shfl_xor(cost, dlt);
            const uint32_t on = (uint32_t)__shfl_xor((int)shares, dlt);
            if (oc < cost || (oc == cost && on < shares)) {
                cost = oc;
                shares = on;
            }
        }
        shares = (uint32_t)uniform((int)shares);
    }
    const uint32_t unit = wg / shares;
    if (unit >= total) return false;
    uint32_t before = 0;
    for (int b0 = 0;; b0 += 64) {
        const uint32_t own = b0 + lane < blocks ? (uint32_t)weight(b0 + lane) : 0u;
        uint32_t upto = own;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const uint32_t v = (uint32_t)__shfl_up((int)upto, dlt);
            if (lane >= dlt) upto += v;
        }
        const uint64_t past = __ballot(before + upto > unit);
        if (past != 0ull) {
            const int l = __ffsll((unsigned long long)past) - 1;
            s.block = b0 + l;
            s.nth = uniform((int)(unit - before) - __shfl((int)(upto - own), l));
            s.share = (int)(wg - unit * shares);
            s.shares = (int)shares;
            return true;
        }
        before += (uint32_t)__shfl((int)upto, 63);
        if (b0 + 64 >= blocks) return false;  // (not reached: the last unit is below the total)
    }
}

// ------------------------------------------------------------------------------------------------
// The filter pass of the LDS-resident search on 16-bit tables (option lds_filter = 2).
//     The pass that looks at every encoding only has to decide which ones can be among the k nearest; it is bound by
//     the LDS reads of table entries.  Here an entry is two bytes: scaled so that the query's bound becomes
//     2^(C-1), truncated, and cut off at 2^C - 1, with C = 13 for M = 8 and 12 for M = 16 chunks, so that the sum of
//     M entries fits 16 bits.  A sub-tile then holds twice the queries in the same LDS (32 at M = 8), a lane's
//     16-byte read serves 8 queries, and a packed 16-bit add two of them: half the LDS reads and about two thirds
//     of the vector instructions per distance.  Truncation makes a sum too small by at most M units, never too
//     large, and the bound is rounded up: no encoding whose float32 distance is at or below the bound is lost; a
//     share of M / 2^(C-1) of the bound's neighbourhood comes along.  k_select keeps what lies within the rounding
//     of the k-th smallest sum and recomputes those distances as float32 sums of the float32 tables, which is what
//     is ordered and returned (see SelectArgs::fx_margin).
//     Geometry, item walk, distance context and line layout are those of k_lds<G> (rows of 64 or 32 bytes, lines
//     of 256 bytes, chunk order rotated per lane group); a sub-tile has 128 / G queries.
//     WALK_KEPT: the blocks of 64 encodings that a sub-tile's list names, unit after unit of the work that k_units has cut.  The next
//     block's records are requested a block ahead (without that, and with the units cut here instead of in a launch, which cost 79
//     scalar registers too many, it ran at 0.6 of this rate).  At M = 8 it looks at 0.7 of the pairs a second that the walk of
//     everything does (10 000 queries on 700 000 encodings: 0.40 ms for 0.21 of them, 1.31 for all): a step takes 44 clocks of the
//     LDS pipe in place of 39 and 42 vector instructions in place of 34 (neighbours of a list are not neighbours in the tree: the
//     context helps less; and every unit stages its tables), and the pipe is busy 0.55
//     of the time in place of 0.66, with half as many waits again (units begin and end).  At M = 16, without the context, 0.67 of
//     the pipe's time, 2.5 ms for 0.114 of 6.5 million encodings.
//     WALK_NEAR: the least sums of the nearest blocks, for k_tau.  0.27 of the pipe's time at M = 8: 313 workgroups in two rounds of 256.
//     grid (blocks, G / 2, tiles), or, behind k_mm16, (workgroups) for the sub-tiles of the blocks that it has not done
//     (find_share), or (256) for WALK_KEPT, (sub-tiles, workgroups per sub-tile) for WALK_NEAR; block 1024, dynamic LDS
//     lds_table_bytes(G) + lds16_aux_bytes(); G in {4, 8}.
// ------------------------------------------------------------------------------------------------
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) const u16x8 lds_u16x8_t;

__host__ __device__ constexpr int fx16_cap_bits(int M) { return M <= 4 ? 14 : M <= 8 ? 13 : 12; }

enum { WALK_ALL = 0, WALK_KEPT = 1, WALK_NEAR = 2 };
struct ListArgs {
    const uint16_t *list;   // [sub-tiles][nblk] kept blocks of 2^shift x 64 encodings (k_prune): all of them in any order, or, first, the nearest
                            // classes and behind them the next one
    int nblk, shift;
    const uint4 *units;     // WALK_KEPT: sub-tile, part of its list
    uint32_t *state;        // WALK_KEPT: the number of units, the next one to take
    const uint4 *near;      // WALK_NEAR: [sub-tiles] blocks of the list to take all of, the number of those to take some of, how many of them
    const uint32_t *ebegin; // WALK_NEAR: id range of every encoding
    float *gmin;            // WALK_NEAR: [tiles*64][gstride] a query's minima, one for each of 64 positions in a block and wave
    int64_t gstride;
};

template <int G, int M4, bool CTX, int WALK = WALK_ALL>
__global__ __launch_bounds__(1024) void k_lds16(const uint32_t *__restrict__ rec, int64_t nitems, const float *__restrict__ lutT,
                                                int K, int per_block, OutArgs o, ListArgs la)
{
    constexpr int M = 4 * M4, Qs = 2 * WAVE / G, V = 8, LPI = Qs / V, IPS = WAVE / LPI;
    constexpr int CPL = lds_chunks_per_line(G), NG = M / CPL, U = M4 >= 4 ? 2 : 4, RING = LDS16_RING;
    constexpr int CB = fx16_cap_bits(M);
    constexpr uint32_t CAP = (1u << CB) - 1u;
    constexpr float TOP = (float)(1u << (CB - 1));
    static_assert(CPL * Qs * 2 == 256 && (G == 4 || G == 8), "lines of 256 bytes");
    extern __shared__ float lds[];
    constexpr uint32_t rowB = Qs * 2, lineB = CPL * rowB, KP = 256;
    char *aux = reinterpret_cast<char *>(lds) + (size_t)NG * KP * lineB;
    typedef uint32_t u32v4 __attribute__((ext_vector_type(4)));
    u32v4(*ringx)[RING] = reinterpret_cast<u32v4(*)[RING]>(aux);
    uint32_t(*ringm)[RING] = reinterpret_cast<uint32_t(*)[RING]>(aux + 16 * RING * 16);
    uint32_t(*wcount)[64] = reinterpret_cast<uint32_t(*)[64]>(aux + 16 * RING * 20);
    uint32_t(*wpos)[64] = reinterpret_cast<uint32_t(*)[64]>(aux + 16 * RING * 20 + 16 * 64 * 4);
    int tile = blockIdx.z, sub = blockIdx.y, share = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int w = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
    constexpr bool LIST = WALK != WALK_ALL;
    uint4 near = make_uint4(0u, 0u, 0u, 0u);
    uint32_t from = 0u, to = 0u, cs = 0u;  // the part of the list of sub-tile cs
    for (;;) {  // (once, or once per unit)
    if (WALK == WALK_KEPT) {
        uint32_t *ticket = reinterpret_cast<uint32_t *>(aux + 16 * RING * 20 + 2 * 16 * 64 * 4);
        if (threadIdx.x == 0) *ticket = atomicAdd(&la.state[1], 1u);
        __syncthreads();
        const uint32_t u = (uint32_t)uniform((int)*ticket);
        if (u >= la.state[0]) return;
        const uint4 unit = la.units[u];
        cs = (uint32_t)uniform((int)unit.x);
        from = (uint32_t)uniform((int)unit.y);
        to = (uint32_t)uniform((int)unit.z);
        tile = (int)cs / (QT / Qs);
        sub = (int)cs % (QT / Qs);
    } else if (WALK == WALK_NEAR) {
        cs = blockIdx.x;
        tile = (int)cs / (QT / Qs);
        sub = (int)cs % (QT / Qs);
        near = la.near[cs];
        to = near.x + near.z;
    } else if (o.done) {
        const uint32_t taken = o.done[2 * o.blocks];
        if (taken == (uint32_t)o.blocks) return;
        // a sub-tile of Qs queries: the nth of its block's that hold a query
        Share s = {0, (int)blockIdx.x / o.shares, (int)blockIdx.x % o.shares, o.shares};
        if (taken != 0u &&
            !find_share(blockIdx.x, gridDim.x, o.blocks, nitems, o.fixed ? o.shares : 0,
                        [&](int b) { return o.done[b] != 0u ? 0 : (int)((min<int64_t>(MM_Q, o.nq - (int64_t)b * MM_Q) + Qs - 1) / Qs); }, s))
            return;
        tile = s.block * (MM_Q / QT) + s.nth / (QT / Qs);  // (all of them: numbered through)
        sub = s.nth % (QT / Qs);
        share = s.share;
        per_block = (int)((nitems + s.shares - 1) / s.shares);
    }
    wcount[w][lane] = 0u;
    // ---- stage the sub-tile's tables as 16-bit entries: piece p of row (m, k) holds queries 8p .. 8p+7
    {
        constexpr int P8 = Qs / 8;
        const int p = (int)threadIdx.x % P8;  // the block size is a multiple of P8: a thread always converts the same queries
        float sc[8];
        bool dead[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const float t = o.tau[(int64_t)tile * QT + sub * Qs + p * 8 + v];
            dead[v] = !(t >= 0.f);
            sc[v] = TOP / fmaxf(t, 8.0779e-28f);
        }
        const float *src = lutT + (int64_t)tile * M * K * QT + sub * Qs + p * 8;
        const int total = M * K * P8;
        for (int idx0 = 0; idx0 < total; idx0 += (int)blockDim.x * 4) {
            float4 a[4][2];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = idx0 + u * (int)blockDim.x + (int)threadIdx.x;
                const int row = min(idx, total - 1) / P8;
                a[u][0] = *reinterpret_cast<const float4 *>(src + (int64_t)row * QT);
                a[u][1] = *reinterpret_cast<const float4 *>(src + (int64_t)row * QT + 4);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = idx0 + u * (int)blockDim.x + (int)threadIdx.x;
                if (idx >= total) break;
                const int row = idx / P8;
                const int m = K == 256 ? row >> 8 : row / K, k = row - m * K;
                const float e[8] = {a[u][0].x, a[u][0].y, a[u][0].z, a[u][0].w, a[u][1].x, a[u][1].y, a[u][1].z, a[u][1].w};
                uint32_t q[8];
#pragma unroll
                for (int v = 0; v < 8; ++v) q[v] = dead[v] ? CAP : min((uint32_t)fminf(e[v] * sc[v], (float)CAP), CAP);
                uint4 pk;
                pk.x = q[0] | (q[1] << 16);
                pk.y = q[2] | (q[3] << 16);
                pk.z = q[4] | (q[5] << 16);
                pk.w = q[6] | (q[7] << 16);
                *reinterpret_cast<uint4 *>(reinterpret_cast<char *>(lds) + (size_t)(((m / CPL) * KP + k) * CPL + (m % CPL)) * rowB + p * 16) = pk;
            }
        }
        __syncthreads();
    }
    const int lg = lane / LPI, lq = lane % LPI;
    const int col = sub * Qs + lq * V;  // first of this lane's queries inside the tile
    const int jr = lg & (CPL - 1);
    uint32_t sh[2][CPL], pb[NG][CPL];
#pragma unroll
    for (int t = 0; t < CPL; ++t) {
        int c0 = t ^ jr;
        if (CTX) c0 = t < 4 ? (t ^ (jr & 1)) : 4 + ((t - 4) ^ (jr & 3));
        const int c1 = t ^ jr;
        sh[0][t] = 0x03020000u | ((4u + (uint32_t)(c0 & 3)) << 8);
        sh[1][t] = 0x03020000u | ((4u + (uint32_t)(c1 & 3)) << 8);
#pragma unroll
        for (int g = 0; g < NG; ++g) pb[g][t] = (uint32_t)(lq * 16) + (uint32_t)g * KP * lineB + (uint32_t)(g == 0 ? c0 : c1) * rowB;
    }
    const bool cross = CPL == 8 && (jr & 4) != 0;
    // a lane's 16 bytes are eight 16-bit entries, added as four dwords: no half can carry into its neighbour because
    // a sum of M capped entries stays below 2^16, and three dwords add in one instruction
    typedef __attribute__((address_space(3))) const u32v4 lds_u32v4_t;
    auto look = [&](const uint32_t dw[M4], int g, int t) -> u32v4 {
        uint32_t src;
        if (CPL == 4) {
            src = dw[g];
        } else {
            const bool second = (CTX && g == 0) ? t >= 4 : ((t >= 4) != cross);
            src = second ? dw[2 * g + 1] : dw[2 * g];
        }
        return *reinterpret_cast<lds_u32v4_t *>(__builtin_amdgcn_perm(src, pb[g][t], sh[g == 0 ? 0 : 1][t]));
    };
    const int64_t blo = LIST ? 0 : (int64_t)share * per_block;
    const int64_t bhi = min(nitems, blo + per_block);
    // the largest sum that may pass, plus one, per query of this lane
    u16x8 tp1;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const float t = o.tau[(int64_t)tile * QT + col + v];
        const float scale = TOP / fmaxf(t, 8.0779e-28f);
        tp1[v] = (t >= 0.f) ? (unsigned short)(min((uint32_t)fminf(t * scale * (1.f + 1.9073486e-6f), 60000.f), 60000u) + 2u) : (unsigned short)0;
    }
    // Candidates.  x holds, per query of the lane, bound + 1 - sum where the sum is at or below the bound, else 0 (four
    // dwords of two halves).  The loop over the items only parks what it finds: a lane with a non-zero half puts all of x
    // and (its lane number, the item) into the wave's ring, slot = its rank among such lanes.  When the next step's
    // entries might not fit, the wave takes the ring apart, all lanes at once: the non-zero halves are counted per
    // query (LDS atomics), the wave reserves that many slots of each query's list with one global atomic per query,
    // and every half is written as (sum, item), the sum being its owner's bound + 1 minus the half.
    const u32v4 tp1w = __builtin_bit_cast(u32v4, tp1);
    int held = 0;
    auto flush = [&]() {
        auto each_half = [&](auto f) {
            for (int base = 0; base < held; base += 64) {  // every lane goes round: the bounds come from other lanes
                const bool valid = base + lane < held;
                const int i = valid ? base + lane : 0;
                const u32v4 x = ringx[w][i];
                const uint32_t meta = ringm[w][i];
                const int src = (int)(meta >> 26);
                const int c0 = sub * Qs + (src % LPI) * V;  // the owner's first query inside the tile
                u32v4 t;
                t.x = (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)tp1w.x);
                t.y = (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)tp1w.y);
                t.z = (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)tp1w.z);
                t.w = (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)tp1w.w);
#pragma unroll
                for (int h = 0; h < 8; ++h) {
                    const uint32_t xh = (x[h >> 1] >> (16 * (h & 1))) & 0xFFFFu;
                    const uint32_t th = (t[h >> 1] >> (16 * (h & 1))) & 0xFFFFu;
                    if (valid && xh != 0u) f(c0 + h, th - xh, meta & 0x3FFFFFFu);
                }
            }
        };
        each_half([&](int c, uint32_t, uint32_t) { atomicAdd(&wcount[w][c], 1u); });
        __builtin_amdgcn_wave_barrier();
        const uint32_t cq = wcount[w][lane];
        wpos[w][lane] = cq ? atomicAdd(&o.cnt[(int64_t)tile * QT + lane], cq) : 0u;
        wcount[w][lane] = 0u;
        __builtin_amdgcn_wave_barrier();
        each_half([&](int c, uint32_t val, uint32_t rel) {
            const uint32_t pos = atomicAdd(&wpos[w][c], 1u);
            if (pos < o.C) o.cand[((int64_t)tile * QT + c) * o.C + pos] = ((uint64_t)val << 32) | (uint32_t)(blo + (int64_t)rel);
        });
        __builtin_amdgcn_wave_barrier();
        held = 0;
    };
    auto emit = [&](const u32v4 &x, uint64_t bal, uint32_t rel) {
        const int n = __popcll(bal);
        if (held + n > RING) flush();
        if (((x.x | x.y) | (x.z | x.w)) != 0u) {
            const int slot = held + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            ringx[w][slot] = x;
            ringm[w][slot] = ((uint32_t)lane << 26) | rel;
        }
        held += n;
    };
    uint32_t prev0 = 0u;
    u32v4 top = 0u;
    // U steps of the wave: records dw, step u live in this lane if alive(u) (`whole`: in all lanes); item(u) is the item's number,
    // `start` the walk's first step.  (The walk of a list has one copy of this: two of them spill at M = 16.)
    auto evaluate = [&](const uint32_t (&dw)[U][M4], bool start, bool whole, auto check, auto alive, auto item) {
        constexpr bool CHECK = decltype(check)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = !CHECK || alive(u);
            bool fast = false;
            if (CTX) {
                const bool differs = live && ((dw[u][0] ^ prev0) & 0xFFFFu) != 0u;
                fast = __ballot(differs) == 0ull && !(start && u == 0);
                prev0 = dw[u][0];
            }
            if (!CTX || !fast) top = look(dw[u], 0, 0) + look(dw[u], 0, 1);
            u32v4 d = top;
            {
                // the remaining M - 2 entries, two at a time
                u32v4 e[M - 2];
#pragma unroll
                for (int j = 2; j < M; ++j) e[j - 2] = look(dw[u], j / CPL, j % CPL);
#pragma unroll
                for (int j = 0; j < M - 2; j += 2) d = d + e[j] + e[j + 1];
            }
            // a sum at or below its bound: (bound + 1) - sum, saturating at zero, is not zero
            u32v4 x = __builtin_bit_cast(u32v4, __builtin_elementwise_sub_sat(tp1, __builtin_bit_cast(u16x8, d)));
            if (CHECK && !live) x = 0u;
            if (LIST && !whole) {
                asm volatile("" ::: "memory");  // (a branch, not four selects in every step)
                if (!alive(u)) x = 0u;
            }
            const uint64_t bal = __ballot(((x.x | x.y) | (x.z | x.w)) != 0u);
            if (bal != 0ull) emit(x, bal, item(u));
        }
    };
    if constexpr (LIST) {
        static_assert(U * IPS == 64, "a block of 64 is one round of the walk");
        const uint16_t *list = la.list + (int64_t)cs * la.nblk;
        const rsrc_t rr = make_rsrc(rec, (uint32_t)(nitems * (M4 * 4)));
        const uint32_t voff = (uint32_t)lg * (M4 * 4);
        // The block of 64 from item `at` on; at the index's end its last 64, of which those below `at` have had their turn.  The records
        // of the next block are requested before this one's are looked up.
        auto first_of = [&](uint32_t at) { return min(at, (uint32_t)nitems - 64u); };
        auto load = [&](uint32_t (&dw)[U][M4], uint32_t at) {
            const uint32_t base = first_of(at);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k2 = 0; k2 < M4; ++k2)
                    dw[u][k2] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rr, (int)voff + 4 * k2, (int)((base + u * IPS) * (M4 * 4)), 0);
        };
        uint32_t dw[U][M4], nx[U][M4];
        if constexpr (WALK == WALK_KEPT) {
            // a wave takes a run of the part's blocks of 64 encodings; the numbers of the next 64 kept blocks lie in its lanes
            const uint32_t n64 = (to - from) << la.shift;
            const uint32_t i0 = n64 * (uint32_t)w / 16u, i1 = n64 * (uint32_t)(w + 1) / 16u;
            uint32_t held_from = from + (i0 >> la.shift), held_blk = list[min(held_from + (uint32_t)lane, to - 1u)];
            auto block_at = [&](uint32_t i) -> uint32_t {
                const uint32_t e = from + (i >> la.shift);
                if (e - held_from == 64u) {
                    held_from = e;
                    held_blk = list[min(e + (uint32_t)lane, to - 1u)];
                }
                const uint32_t blk = (uint32_t)__builtin_amdgcn_readlane((int)held_blk, (int)(e - held_from));
                return ((blk << la.shift) + (i & ((1u << la.shift) - 1u))) << 6;
            };
            if (i0 < i1) {
                uint32_t at = block_at(i0);
                load(dw, at);
                for (uint32_t i = i0; i < i1; ++i) {
                    const uint32_t next = block_at(min(i + 1u, i1 - 1u));
                    load(nx, next);
                    const uint32_t base = first_of(at);
                    auto item = [&](int u) { return base + (uint32_t)(u * IPS + lg); };
                    evaluate(dw, i == i0, base == at, std::false_type{}, [&](int u) { return item(u) >= at; }, item);
                    at = next;
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int k2 = 0; k2 < M4; ++k2) dw[u][k2] = nx[u][k2];
                }
            }
            flush();
            __syncthreads();
            continue;
        } else {
            // The least sum of every position in a block, over the blocks of 64 that this wave takes: neighbours in the index go to
            // different minima.  The low four bits of a sum make room for how many vectors have the encoding, as 15 - log2: the k-th
            // nearest vector is what has to be bounded, and a small tight cluster may have fewer than k encodings.  A sum with an
            // entry that was cut off is at least CAP: no bound.  Otherwise the encoding's distance is at most the sum, rounded up,
            // and one unit for every entry's truncation, over the scale.
            const rsrc_t re = make_rsrc(la.ebegin, (uint32_t)((nitems + 1) * 4));
            uint32_t eb[U], nb[U];  // how many, of this block and of the next
            auto load_many = [&](uint32_t (&many)[U], uint32_t at) {
                const uint32_t base = first_of(at);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    many[u] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(re, lg * 4 + 4, (int)((base + u * IPS) * 4), 0) -
                              (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(re, lg * 4, (int)((base + u * IPS) * 4), 0);
            };
            const uint32_t waves = gridDim.y * 16u, g = blockIdx.y * 16u + (uint32_t)w, n64 = to << la.shift;
            u16x8 lo[U];
#pragma unroll
            for (int u = 0; u < U; ++u) lo[u] = (unsigned short)0xFFFFu;
            // this wave's j-th block of 64 is number g + j waves; the numbers of the next 64 lie in its lanes
            const uint32_t mine = g < n64 ? (n64 - g + waves - 1u) / waves : 0u;
            uint32_t held = 0u;
            auto block_at = [&](uint32_t j) -> uint32_t {
                if ((j & 63u) == 0u) {
                    const uint32_t i = min(g + (j + (uint32_t)lane) * waves, n64 - 1u);
                    uint32_t e = i >> la.shift;
                    if (e >= near.x) e = near.x + (uint32_t)((uint64_t)(e - near.x) * near.y / near.z);
                    held = (((uint32_t)list[e] << la.shift) + (i & ((1u << la.shift) - 1u))) << 6;
                }
                return (uint32_t)__builtin_amdgcn_readlane((int)held, (int)(j & 63u));
            };
            if (mine != 0u) {
                uint32_t at = block_at(0u);
                load(dw, at);
                load_many(eb, at);
                for (uint32_t j = 0; j < mine; ++j) {
                    const uint32_t next = j + 1u < mine ? block_at(j + 1u) : at;
                    load(nx, next);
                    load_many(nb, next);
                    const uint32_t base = first_of(at);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        u32v4 e[M - 2], d = look(dw[u], 0, 0) + look(dw[u], 0, 1);
#pragma unroll
                        for (int c = 2; c < M; ++c) e[c - 2] = look(dw[u], c / CPL, c % CPL);
#pragma unroll
                        for (int c = 0; c < M - 2; c += 2) d = d + e[c] + e[c + 1];
                        d = (d | 0x000F000Fu) - min(31u - (uint32_t)__builtin_clz(eb[u] | 1u), 15u) * 0x00010001u;
                        if (base != at && base + (uint32_t)(u * IPS + lg) < at) d = 0xFFFFFFFFu;  // (another block's: an encoding counts once)
                        lo[u] = __builtin_elementwise_min(lo[u], __builtin_bit_cast(u16x8, d));
                    }
                    at = next;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        eb[u] = nb[u];
#pragma unroll
                        for (int k2 = 0; k2 < M4; ++k2) dw[u][k2] = nx[u][k2];
                    }
                }
            }
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const float t = o.tau[(int64_t)tile * QT + col + v], scale = TOP / fmaxf(t, 8.0779e-28f);
                float *row = la.gmin + ((int64_t)tile * QT + col + v) * la.gstride + g * 64u;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t raw = lo[u][v], top = raw | 15u;
                    // (log2 of how many in the low four bits of the number too)
                    const uint32_t bits = (__float_as_uint((float)(top + M + 1) / scale * (1.f + 1.9073486e-6f)) + 15u) & ~15u;
                    row[u * IPS + lg] = __uint_as_float(top < CAP && bits < 0x7F800000u ? bits | (15u - (raw & 15u)) : 0x7F800000u);
                }
            }
            return;
        }
    } else {
    constexpr int RF = IPS;
    if (blo >= bhi) return;
    const int nruns = nw * IPS / RF;
    const int RLr = (per_block + nruns - 1) / nruns;
    const int RL = (RLr + RF - 1) / RF;
    const int ph = lg % RF;
    const int64_t rlo = blo + (int64_t)((w * IPS + lg) / RF) * RLr;
    const int runlen = (int)max<int64_t>(0, min<int64_t>(bhi - rlo, RLr));
    const int len = runlen > ph ? (runlen - ph + RF - 1) / RF : 0;
    int minlen = len;
#pragma unroll
    for (int dlt = LPI; dlt < WAVE; dlt <<= 1) minlen = min(minlen, __shfl_xor(minlen, dlt));
    minlen = uniform(minlen);
    const rsrc_t rr = make_rsrc(rec + blo * M4, (uint32_t)((bhi - blo) * (M4 * 4)));
    const uint32_t first = (uint32_t)(rlo - blo) + (uint32_t)ph;
    const uint32_t voff = len > 0 ? first * (M4 * 4) : 0u;
    auto steps = [&](int i, auto check) {
        constexpr bool CHECK = decltype(check)::value;
        uint32_t dw[U][M4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t vo = voff;
            int so = (i + u) * (RF * M4 * 4);
            if (CHECK) {
                vo += (uint32_t)max(0, min(i + u, len - 1)) * (RF * M4 * 4);
                so = 0;
            }
#pragma unroll
            for (int k2 = 0; k2 < M4; ++k2) dw[u][k2] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rr, (int)vo + 4 * k2, so, 0);
        }
        evaluate(dw, i == 0, !CHECK, check, [&](int u) { return i + u < len; }, [&](int u) { return first + (uint32_t)(i + u) * RF; });
    };
    int i = 0;
    for (; i + U <= minlen; i += U) steps(i, std::false_type{});
    for (; i < RL; i += U) steps(i, std::true_type{});
    flush();
    return;
    }
    }
}

// ------------------------------------------------------------------------------------------------
// The filter pass of the search on the matrix cores (few dimensions per chunk).
//     For the decision "can this encoding be among the k nearest" the distance may also be taken as what it is, the
//     distance to the encoding's reconstruction r: ||q - r||^2 = ||q||^2 - 2 (q.r - ||r||^2 / 2), a contraction over the
//     dimensions in 16-bit floats.  A lane's operand for 8 dimensions of an encoding is a 16-byte piece of a codeword,
//     read from LDS at the code: no tables, no staged reconstruction, and one read serves 128 queries.  All codewords
//     in 16 bits (32 dpad bytes per code value: 64 KB at 128 dimensions) are staged once per workgroup; a wave keeps the
//     operands of 128 queries in registers and walks 32 encodings per step.  The walk then costs dpad / 16 matrix
//     instructions per 32 x 32 distances however many chunks an encoding has, where k_lds16 reads M table entries.
//     Exactness.  Queries and codewords are taken relative to the codebooks' means, scaled by powers of two (codewords
//     by one for all, queries by one per workgroup).  With q = q^ + e, c = c^ + f (q^, c^ the 16-bit values; nothing is
//     assumed of the conversion: e and f are computed) the error of a chunk's product is e.c^ + q^.f + e.f.  The
//     first two are evaluated here for every (query, chunk, codeword), on the matrix cores again, and the largest of a chunk
//     taken: their sum over the chunks is half of what sqrt(sum ||e||^2) sqrt(sum ||c||^2) and its like would give.
//     Everything else is float32 rounding: in units of 2^-24
//     (||q||^2 + C^2), C^2 the sum of the largest ||c||^2, the contraction (one unit in the last place per product)
//     4 dpad + 16, ||q||^2 d, the table entries that the float32 distance is summed from 4 ds + 10, the sums of M terms
//     3 M, the centring 4, e and f in 16 bits where their products cancel 8 (2^-11 of sum |e c^| + |q^ f|, each at most 2^-11
//     of sum |q c|): below 6 dpad + 4 ds + 4 M + 64.  E bounds the difference between the value here and the float32
//     distance of the tables, and everything with a value of at most tau + E passes.  Its candidates carry a 16-bit fixed-point
//     value; k_select takes everything within margin = 2 E of the k-th smallest and recomputes those from the tables.
//     Where E is not small against the bound (tight clusters far from the mean), or the sample has so many encodings just above
//     the bound that those up to tau + E would not fit the candidate list (`room`, from k_tau), a block of 128 queries with
//     such a query is left to k_lds16, which is launched behind and otherwise ends at once: where k_tau sees it (`loose`) no
//     workgroup takes the block, where it is found here all of its workgroups end.  The two share a batch from half of its blocks
//     on; below that the second start costs more than the faster rate gives.  Ten million vectors of 16 chunks, 10 000
//     queries (79 blocks) of which 1, 19 and 39 blocks are left: 15.4, 17.5 and 19.3 ms, k_lds16 alone 21.8 (M = 8, 4000
//     queries, half: 2.74 and 2.82).
//     What bounds it: the matrix cores under the card's power limit.  Ten million vectors of 16 chunks (128 dimensions), 6.6
//     million distinct encodings, 10 000 queries: 13.1 ms = 1.29 PFLOP/s, against 1.55 of the bare instruction on random operands and 1.16 to 1.21 of a large
//     library product here; k_lds16 19.7 ms.
//     Candidates: a lane that finds one among its 16 values parks all 16 in the wave's ring; a full ring is taken apart by
//     all lanes (as in k_lds16).
//     MC: chunks, each of at most 8 dimensions (a lane's operand is one chunk's codeword).
//     grid (workgroups) for the blocks that k_tau has left (find_share), block 512, dynamic LDS mm_lds_bytes(MC).
// ------------------------------------------------------------------------------------------------
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
constexpr int MM_RING = 128, MM_WAVES = 8;
__host__ __device__ constexpr size_t mm_lds_bytes(int MC)
{
    return (size_t)MC * 5120 + (size_t)MM_WAVES * MM_RING * 68 + (size_t)MM_WAVES * MM_Q * 8 + MM_Q * 16 + 2 * 64 + 64;
}

struct MmArgs {
    const float *queries;  // rows of this batch
    int64_t nq, nql;       // live queries, queries with state (multiple of 64)
    int d, ds, dsp, K;
    const float *cbc, *cbnorm, *cbmean;  // centred codewords [M][K][dsp], their squared norms, the means [M][ds]
    ChunkOrder ord;
    const float *room;     // [nql] from k_tau: the largest error bound with which the candidates still fit
    const uint32_t *loose; // [blocks] from k_tau: not zero where a query's error bound will exceed that
    uint32_t *margin;      // [nql] for k_select: those of the blocks filtered here are written
    uint32_t *taken;       // count of the blocks that it filtered (etf_last_matrix_blocks)
};

template <int MC>
__global__ __launch_bounds__(512, 2) void k_mm16(const uint32_t *__restrict__ rec, int64_t nitems, OutArgs o, MmArgs a)
{
    constexpr int M4 = MC / 4, KS = MC / 2, NB = MM_Q / 32, RING = MM_RING, NW = MM_WAVES;
    extern __shared__ __align__(16) char mm_raw[];
    f16x8 *piece = reinterpret_cast<f16x8 *>(mm_raw);                                     // [MC][256]
    float *hn = reinterpret_cast<float *>(mm_raw + (size_t)MC * 4096);                    // [MC][256] -||c||^2 / 2, scaled
    char *behind = mm_raw + (size_t)MC * 4096 + (size_t)MC * 1024;
    f16x8 *bstage = reinterpret_cast<f16x8 *>(behind);                                    // [NB][KS][64], before the ring is in use
    f16x8 *estage = bstage + NB * KS * 64;                                                // ... and what the conversion lost, times 2^11
    static_assert((size_t)2 * NB * KS * 64 * 16 <= (size_t)NW * RING * 68, "the staging area lies where the rings will");
    floatx4_t(*ringx)[4][RING] = reinterpret_cast<floatx4_t(*)[4][RING]>(behind);
    uint32_t(*ringm)[RING] = reinterpret_cast<uint32_t(*)[RING]>(behind + NW * RING * 64);
    behind += NW * RING * 68;
    uint32_t(*wcount)[MM_Q] = reinterpret_cast<uint32_t(*)[MM_Q]>(behind);
    uint32_t(*wpos)[MM_Q] = reinterpret_cast<uint32_t(*)[MM_Q]>(behind + NW * MM_Q * 4);
    float(*part)[MM_Q] = reinterpret_cast<float(*)[MM_Q]>(behind);                        // partial sums, before the counters are in use
    behind += NW * MM_Q * 8;
    float4 *qc = reinterpret_cast<float4 *>(behind);                                      // [MM_Q] threshold, offset, factor
    uint32_t *cmax = reinterpret_cast<uint32_t *>(behind + MM_Q * 16);                    // [MC] largest ||c||^2, then of ||f||^2
    uint32_t *fmaxs = cmax + 16, *shared = cmax + 32;                  // shared: max |q|, blocks too loose
    const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int K = a.K, ds = a.ds;
    const float inf = __uint_as_float(0x7F800000u);
    int left = 0;
    for (int b0 = 0; b0 < o.blocks; b0 += 64) left += __popcll(__ballot(b0 + lane < o.blocks && a.loose[b0 + lane] != 0u));
    if (2 * left > o.blocks) return;
    Share sh = {(int)blockIdx.x / o.shares, 0, (int)blockIdx.x % o.shares, o.shares};
    if (left != 0 &&
        !find_share(blockIdx.x, gridDim.x, o.blocks, nitems, o.fixed ? o.shares : 0, [&](int b) { return a.loose[b] != 0u ? 0 : 1; }, sh))
        return;
    const int qb = sh.block;
    const int per_block = (int)((nitems + sh.shares - 1) / sh.shares + 31) / 32 * 32;
    // ---- the largest norms
    if (threadIdx.x < 48) cmax[threadIdx.x] = 0u;
    __syncthreads();
    for (int idx = threadIdx.x; idx < MC * 256; idx += 512) {
        const int m = idx >> 8, k = idx & 255;
        if (k < K) atomicMax(&cmax[m], __float_as_uint(a.cbnorm[(int64_t)a.ord.src[m] * K + k]) & 0x7FFFFFFFu);
    }
    // ---- this wave's share of the queries: block w % 4, one half of the contraction
    static_assert(NB == 4 && NW == 8, "eight waves prepare four blocks of 32 queries");
    const int pbk = w & 3, s0 = (w >> 2) * (KS / 2);
    float qv[KS / 2][8];
    {
        const int64_t ql = (int64_t)qb * MM_Q + pbk * 32 + col;
        const bool live = ql < a.nq;
        const float *row = a.queries + (live ? ql : 0) * a.d;
        const bool wide = (ds & 3) == 0 && (a.d & 3) == 0 && ((reinterpret_cast<uintptr_t>(a.queries) | reinterpret_cast<uintptr_t>(a.cbmean)) & 15) == 0;
        float mx = 0.f, nn = 0.f;
#pragma unroll
        for (int s = 0; s < KS / 2; ++s) {
            const int src = a.ord.src[2 * (s0 + s) + half];
            if (wide) {
#pragma unroll
                for (int i = 0; i < 8; i += 4) {
                    float4 v = make_float4(0.f, 0.f, 0.f, 0.f), u = v;
                    if (live && i < ds) {
                        v = *reinterpret_cast<const float4 *>(row + src * ds + i);
                        u = *reinterpret_cast<const float4 *>(a.cbmean + src * ds + i);
                    }
                    qv[s][i] = v.x - u.x;
                    qv[s][i + 1] = v.y - u.y;
                    qv[s][i + 2] = v.z - u.z;
                    qv[s][i + 3] = v.w - u.w;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) qv[s][i] = (live && i < ds) ? row[src * ds + i] - a.cbmean[src * ds + i] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                mx = fmaxf(mx, fabsf(qv[s][i]));
                nn = fmaf(qv[s][i], qv[s][i], nn);
            }
        }
        atomicMax(&shared[0], __float_as_uint(mx));
        part[(w >> 2) * 2 + half][pbk * 32 + col] = nn;
    }
    __syncthreads();
    float call = 0.f;
#pragma unroll
    for (int m = 0; m < MC; ++m) call = fmaxf(call, __uint_as_float(cmax[m]));
    // powers of two that bring the largest values to at most 2^14 (values from 2^-14 on keep 11 bits)
    auto scale_for = [](float largest) {
        int e = 0;
        frexpf(fmaxf(largest, 1e-18f), &e);
        return ldexpf(1.f, min(14 - e, 60));
    };
    const float sc = scale_for(sqrtf(call)), sq = scale_for(__uint_as_float(shared[0]));
    const float sigma = sc * sq;
    auto to16 = [](float v) -> _Float16 { return (_Float16)(fabsf(v) < 6.1035156e-5f ? 0.f : v); };  // no subnormal operands
    // ---- codewords as operands
    for (int idx = threadIdx.x; idx < MC * 256; idx += 512) {
        const int m = idx >> 8, k = idx & 255;
        const int64_t src = (int64_t)a.ord.src[m] * K + min(k, K - 1);
        const float *c = a.cbc + src * a.dsp;
        float ff = 0.f;
        f16x8 h;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float v = i < ds ? c[i] : 0.f;
            h[i] = to16(v * sc);
            const float f = v - (float)h[i] / sc;
            ff = fmaf(f, f, ff);
        }
        piece[m * 256 + k] = h;
        hn[m * 256 + k] = -0.5f * sigma * a.cbnorm[src];
        atomicMax(&fmaxs[m], __float_as_uint(ff) & 0x7FFFFFFFu);
    }
    {
        float ee = 0.f;
#pragma unroll
        for (int s = 0; s < KS / 2; ++s) {
            f16x8 h, l;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                h[i] = to16(qv[s][i] * sq);
                const float e = qv[s][i] - (float)h[i] / sq;
                l[i] = to16(e * (2048.f * sq));
                ee = fmaf(e, e, ee);
            }
            bstage[(pbk * KS + s0 + s) * 64 + lane] = h;
            estage[(pbk * KS + s0 + s) * 64 + lane] = l;
        }
        part[4 + (w >> 2) * 2 + half][pbk * 32 + col] = ee;
    }
    __syncthreads();
    // ---- the largest |e.c^ + q^.f| (times 2^11 sigma) of every (query, chunk): wave w takes chunks w and w + 8
    {
        float sum[NB] = {0.f, 0.f, 0.f, 0.f};
        for (int m = w; m < MC; m += NW) {
            const bool mine = half == (m & 1);  // the other half of the contraction is the neighbouring chunk: zeros
            float most[NB] = {0.f, 0.f, 0.f, 0.f};
            for (int t = 0; t * 32 < K; ++t) {
                const int k = t * 32 + col;
                f16x8 h = piece[m * 256 + k], l;
                const float *c = a.cbc + ((int64_t)a.ord.src[m] * K + min(k, K - 1)) * a.dsp;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float v = i < ds ? c[i] : 0.f;
                    l[i] = mine ? to16((v - (float)h[i] / sc) * (2048.f * sc)) : (_Float16)0.f;
                    if (!mine) h[i] = (_Float16)0.f;
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    floatx16 acc;
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(h, estage[(b * KS + (m >> 1)) * 64 + lane], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(l, bstage[(b * KS + (m >> 1)) * 64 + lane], acc, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 16; ++r) most[b] = fmaxf(most[b], fabsf(acc[r]));
                }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) sum[b] += fmaxf(most[b], __shfl_xor(most[b], 32));
        }
        if (half == 0)
#pragma unroll
            for (int b = 0; b < NB; ++b) part[8 + w][b * 32 + col] = sum[b];
    }
    __syncthreads();
    // ---- per query: error bound, threshold, fixed-point form
    if (threadIdx.x < MM_Q) {
        const int t = threadIdx.x;
        const int64_t ql = (int64_t)qb * MM_Q + t;
        const float nq = (part[0][t] + part[1][t]) + (part[2][t] + part[3][t]);
        const float ee = (part[4][t] + part[5][t]) + (part[6][t] + part[7][t]);
        float F = 0.f, C = 0.f, L = 0.f;
        for (int m = 0; m < MC; ++m) {
            F += __uint_as_float(fmaxs[m]);
            C += __uint_as_float(cmax[m]);
        }
#pragma unroll
        for (int i = 0; i < NW; ++i) L += part[8 + i][t];
        // (1.01: the rounding of e and f themselves, and 8 units of G where their products cancel; MC / 32: what to16 dropped of
        // them, two units of 2^-14 per dimension)
        const float G = (float)(6 * 8 * MC + 4 * ds + 4 * MC + 64) * 5.9604645e-8f;
        const float E = 1.01f * (2.f * L * 4.8828125e-4f + (float)MC * 0.03125f) / sigma + 2.02f * sqrtf(ee * F) + G * (nq + C);
        const float tau = ql < a.nql ? o.tau[ql] : -1.f;
        float thr = inf, c0 = 0.f, c1 = 0.f;
        uint32_t margin = 0u;
        if (ql < a.nq && tau >= 0.f) {
            if (!(E <= a.room[ql]) || !(E * 24.f <= tau) || !(tau < inf) || !(sigma * (nq + C) < 1e37f)) atomicMax(&shared[1], 1u);
            const float S = 32000.f / (tau + 2.f * E);
            thr = sigma * (0.5f * (nq - tau) - 0.5f * E);
            c0 = (nq + E) * S;
            c1 = 2.f * S / sigma;
            margin = (uint32_t)fminf(2.002f * E * S + c0 * 9.5367432e-7f + 6.f, 60000.f);
        }
        qc[t] = make_float4(thr, c0, c1, __uint_as_float(margin));
    }
    __syncthreads();
    if (shared[1] != 0u) return;
    if (sh.share == 0) {
        if (threadIdx.x < MM_Q && (int64_t)qb * MM_Q + threadIdx.x < a.nql) a.margin[(int64_t)qb * MM_Q + threadIdx.x] = __float_as_uint(qc[threadIdx.x].w);
        if (threadIdx.x == 0) {
            o.done[qb] = 1u;
            atomicAdd(&o.done[2 * o.blocks], 1u);
            atomicAdd(a.taken, 1u);
        }
    }
    f16x8 B[NB][KS];
    float thr[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int s = 0; s < KS; ++s) B[b][s] = bstage[(b * KS + s) * 64 + lane];
        thr[b] = qc[b * 32 + col].x;
    }
    __syncthreads();  // the staging area becomes the rings and counters
    for (int i = lane; i < MM_Q; i += 64) wcount[w][i] = 0u;
    const int64_t blo = (int64_t)sh.share * per_block, bhi = min(nitems, blo + per_block);
    if (blo >= bhi) return;
    const int live_items = (int)(bhi - blo);
    int held = 0;
    // A full ring: which of an entry's 16 values pass (a mask), how many per query (LDS atomics, which also hand every entry
    // its place among them), one global reservation per query, then the values, nearly always one per entry.
    auto flush = [&]() {
        constexpr int PASS = (RING + 63) / 64;
        uint32_t mask[PASS], at[PASS], meta[PASS];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < PASS; ++u) {
            const int i = u * 64 + lane;
            mask[u] = 0u;
            if (i < held) {
                meta[u] = ringm[w][i];
                const int q = (int)((meta[u] >> 26) & 31u) + 32 * (int)((meta[u] >> 24) & 3u);
                const int left = live_items - (int)(meta[u] & 0xFFFFFFu) * 32 - 4 * (int)(meta[u] >> 31);  // items from the entry's first on
                const float t = qc[q].x;
                uint32_t below = 0u;
#pragma unroll
                for (int g = 3; g >= 0; --g) {
                    const floatx4_t x = ringx[w][g][i];
#pragma unroll
                    for (int r = 3; r >= 0; --r) below = (below << 1) | (x[r] >= t && 8 * g + r < left ? 0u : 1u);
                }
                mask[u] = ~below & 0xFFFFu;
                if (mask[u]) at[u] = atomicAdd(&wcount[w][q], (uint32_t)__popc(mask[u]));
            }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < MM_Q / 64; ++i) {
            const int q = i * 64 + lane;
            const uint32_t n = wcount[w][q];
            wpos[w][q] = n ? atomicAdd(&o.cnt[(int64_t)qb * MM_Q + q], n) : 0u;
            wcount[w][q] = 0u;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < PASS; ++u) {
            const int i = u * 64 + lane;
            if (mask[u]) {
                const int q = (int)((meta[u] >> 26) & 31u) + 32 * (int)((meta[u] >> 24) & 3u);
                const uint32_t item0 = (uint32_t)blo + (meta[u] & 0xFFFFFFu) * 32u + 4u * (meta[u] >> 31);
                const float4 c = qc[q];
                uint32_t pos = wpos[w][q] + at[u];
                uint64_t *list = o.cand + ((int64_t)qb * MM_Q + q) * o.C;
                while (mask[u]) {
                    const int r = __ffs((int)mask[u]) - 1;
                    mask[u] &= mask[u] - 1u;
                    const float x = reinterpret_cast<const float *>(&ringx[w][r >> 2][i])[r & 3];
                    const uint32_t v = (uint32_t)fminf(fmaxf(c.y - c.z * x, 0.f), 65535.f);
                    if (pos < o.C) list[pos] = ((uint64_t)v << 32) | (item0 + 8u * (uint32_t)(r >> 2) + (uint32_t)(r & 3));
                    ++pos;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        held = 0;
    };
    // ---- the walk: 32 encodings per wave and step, the records one step ahead
    const rsrc_t rr = make_rsrc(rec + blo * M4, (uint32_t)live_items * (M4 * 4));
    uint32_t nextw[M4];
    auto fetch = [&](int step) {
#pragma unroll
        for (int i = 0; i < M4; ++i)
            nextw[i] = __builtin_amdgcn_raw_buffer_load_b32(rr, (int)((uint32_t)col * (M4 * 4) + 4u * i), step * (32 * M4 * 4), 0);
    };
    const char *abase = mm_raw + half * 4096;                                     // piece `half` of a pair
    const char *nbase = reinterpret_cast<const char *>(hn) + half * 1024;         // chunk `half` of a pair
    const int steps = (live_items + 31) / 32;
    // -||r||^2 / 2: this half's chunks summed here, the two halves by the matrix instruction, for every column
    uint32_t rot[M4];  // the codes, shifted so that this half's chunk of a pair is in an even byte
    float part_n = 0.f;
    auto ready = [&]() {
        part_n = 0.f;
#pragma unroll
        for (int i = 0; i < M4; ++i) rot[i] = nextw[i] >> (8 * half);
#pragma unroll
        for (int j = 0; j < MC / 2; ++j) part_n += *reinterpret_cast<const float *>(nbase + j * 2048 + __builtin_amdgcn_ubfe(rot[j >> 1], 16 * (j & 1), 8) * 4);
    };
    // the encodings' operands, AHEAD of them on their way: a read takes longer than the four matrix instructions of one
    constexpr int AHEAD = 2;
    f16x8 av[AHEAD];
    auto operand = [&](int s) -> f16x8 {
        return *reinterpret_cast<const f16x8 *>(abase + s * 8192 + __builtin_amdgcn_ubfe(rot[s >> 1], 16 * (s & 1), 8) * 16);
    };
    if (w < steps) {
        fetch(w);
        ready();
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) av[s] = operand(s);
    }
    for (int step = w; step < steps; step += NW) {
        if (step + NW < steps) fetch(step + NW);
        floatx16 zero;
#pragma unroll
        for (int r = 0; r < 16; ++r) zero[r] = 0.f;
        const floatx16 norm = __builtin_amdgcn_mfma_f32_32x32x2f32(part_n, 1.f, zero, 0, 0, 0);
        floatx16 acc[NB];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[s % AHEAD], B[b][s], s == 0 ? norm : acc[b], 0, 0, 0);
            if (s + AHEAD < KS) av[s % AHEAD] = operand(s + AHEAD);
            __builtin_amdgcn_sched_barrier(0);  // in this order
        }
        ready();  // the next step's, beside the matrix instructions and the tests
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) av[s] = operand(s);
        __builtin_amdgcn_sched_barrier(0);
        float t[NB];
        uint64_t bal[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            t[b] = fmaxf(acc[b][0], acc[b][15]);
#pragma unroll
            for (int r = 1; r < 15; r += 2) t[b] = fmaxf(fmaxf(t[b], acc[b][r]), acc[b][r + 1]);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) bal[b] = __ballot(t[b] >= thr[b]);
        for (uint32_t todo = (1u << NB) - 1u;;) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int n = __popcll(bal[b]);
                if ((todo >> b & 1u) == 0u || held + n > RING) continue;
                if (t[b] >= thr[b]) {
                    const int slot = held + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal[b] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal[b], 0u));
#pragma unroll
                    for (int g = 0; g < 4; ++g) ringx[w][g][slot] = floatx4_t{acc[b][4 * g], acc[b][4 * g + 1], acc[b][4 * g + 2], acc[b][4 * g + 3]};
                    ringm[w][slot] = ((uint32_t)lane << 26) | ((uint32_t)b << 24) | (uint32_t)step;
                }
                held += n;
                todo &= ~(1u << b);
            }
            if (todo == 0u) break;
            flush();
        }
    }
    flush();
}

// ------------------------------------------------------------------------------------------------
// S4  forest reduction (paper "Encoding Forests": per-tree result arrays summed per vector):
//     dist(e) = leafp[0][leaf_of[0][e]] + leafp[1][leaf_of[1][e]] + ...   (tree order).
//     Lane = query; a wave walks consecutive items, each item is T coalesced row reads.
//     items: FILTER -> distinct encodings e; SAMPLE -> sample_enc[i]; ALLPAIRS -> input positions n
//     (e = enc_of_pos[n]), written transposed through LDS so that dist[q][n..n+63] is one store.
//     grid (blocks, tiles), block 256.
// ------------------------------------------------------------------------------------------------
struct ReduceArgs {
    const float *leafp[ETF_MAX_M];
    const uint32_t *leaf_of[ETF_MAX_M];  // nullptr: identity (single tree)
    int64_t U[ETF_MAX_M];
    int T;
};

// rows of one item in every tree, fetched by the lane that owns the item in a 64-item chunk.
// The host fills the entries t >= T of ReduceArgs with copies of tree 0, so that every one of the TMAX
// slots is a valid load and the loops below contain no branch (a branch between the row loads makes the
// compiler wait for each load before issuing the next).
template <int TMAX>
__device__ __forceinline__ void reduce_rows(const ReduceArgs &r, uint32_t e, bool live, uint32_t rows[TMAX])
{
#pragma unroll
    for (int t = 0; t < TMAX; ++t) rows[t] = live ? (r.leaf_of[t] ? r.leaf_of[t][e] : e) : 0u;
}

// UB distances at a time for items s0 .. s0+UB-1 of the chunk: all TMAX*UB row loads are issued before
// the first add; trees are added in order (padding slots add +0, which leaves a sum of squares unchanged)
template <int TMAX>
__device__ __forceinline__ void reduce_batch(const ReduceArgs &r, int tile, int lane, const uint32_t my_rows[TMAX],
                                             int s0, int cnt, float d[UB])
{
    float v[UB][TMAX];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
        const int src = min(s0 + u, cnt - 1);
#pragma unroll
        for (int t = 0; t < TMAX; ++t) {
            const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)my_rows[t], src);
            v[u][t] = r.leafp[t][((int64_t)tile * r.U[t] + row) * QT + lane];
        }
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
        d[u] = v[u][0];
#pragma unroll
        for (int t = 1; t < TMAX; ++t) d[u] += (t < r.T) ? v[u][t] : 0.f;
    }
}

template <int MODE, int TMAX>
__global__ __launch_bounds__(256) void k_reduce(ReduceArgs r, int64_t nitems, const uint32_t *__restrict__ map,
                                                int per_wave, OutArgs o)
{
    const int tile = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int w = uniform(threadIdx.x >> 6);
    const int64_t wv = (int64_t)blockIdx.x * 4 + w;
    const int64_t lo = wv * per_wave;
    const int64_t hi = min(nitems, lo + per_wave);
    __shared__ float tbuf[MODE == OUT_ALLPAIRS ? 4 : 1][MODE == OUT_ALLPAIRS ? 64 : 1][65];
    // OUT_FILTER: passing candidates are parked in LDS (STG per lane and wave) and appended to the
    // query's list in one reservation, so the row loads are not interleaved with atomic round trips
    constexpr int STG = 8;
    __shared__ uint64_t stage[MODE == OUT_FILTER ? 4 : 1][MODE == OUT_FILTER ? STG : 1][64];
    int nloc = 0;
    const int64_t ql = (int64_t)tile * QT + lane;
    auto flush = [&]() {
        const uint32_t pos = atomicAdd(&o.cnt[ql], (uint32_t)nloc);
        for (int i = 0; i < nloc; ++i)
            if (pos + i < o.C) o.cand[ql * o.C + pos + i] = stage[w][i][lane];
        nloc = 0;
    };
    float tauv = 0.f, best = __uint_as_float(0x7F800000u);
    if (MODE == OUT_FILTER) tauv = o.tau[ql];
    for (int64_t base = lo; base < hi; base += 64) {
        const int cnt = (int)min<int64_t>(64, hi - base);
        const bool live = lane < cnt;
        const uint32_t e = live ? (MODE == OUT_FILTER ? (uint32_t)(base + lane) : map[base + lane]) : 0u;
        uint32_t my_rows[TMAX];
        reduce_rows<TMAX>(r, e, live, my_rows);
        const float my_tm = (o.term && live) ? o.term[e] : 0.f;  // the leaf term of the item this lane owns
        for (int s0 = 0; s0 < cnt; s0 += UB) {
            float d[UB];
            reduce_batch<TMAX>(r, tile, lane, my_rows, s0, cnt, d);
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                if (s0 + u >= cnt) break;
                d[u] += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_tm), s0 + u));
                if (MODE == OUT_ALLPAIRS) tbuf[w][s0 + u][lane] = d[u];
                else if (MODE == OUT_SAMPLE) best = fminf(best, d[u]);
                else if (d[u] <= tauv) {
                    stage[w][nloc][lane] = ((uint64_t)__float_as_uint(d[u]) << 32) | (uint32_t)(base + s0 + u);
                    if (++nloc == STG) flush();
                }
            }
        }
        if (MODE == OUT_ALLPAIRS) {
            __builtin_amdgcn_wave_barrier();
            for (int qq = 0; qq < 64; ++qq) {
                const int64_t ql = (int64_t)tile * QT + qq;
                if (ql < o.nq && lane < cnt) o.dist[ql * o.N + base + lane] = tbuf[w][lane][qq];
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (MODE == OUT_FILTER && nloc > 0) flush();
    // OUT_SAMPLE: a wave's items are one sample group (per_wave == gsize); keep its minimum
    if (MODE == OUT_SAMPLE && lo < hi) o.gmin[((int64_t)tile * QT + lane) * o.gstride + wv] = best;
}

// ------------------------------------------------------------------------------------------------
// S5a  per-query bound from the sample.  Input: the minimum distance of each of S sample groups.  The
//      k-th smallest group minimum is an upper bound of the k-th smallest database distance, because k
//      different encodings (one per group) are at or below it.
//      A wave per query holds the minima in registers (distances are >= 0, so the bit patterns order like the
//      values) and bisects between the smallest and the largest of them until at most 2^7 patterns are left, 2^-16 of the
//      value: a step is NV compares whose lane masks are counted on the scalar unit, no LDS and no barrier.  (A radix
//      select over LDS histograms of 64 queries per workgroup took 28 us however few queries there were and 32 us
//      for ten thousand, mostly clearing and scanning 64 KB of counters three times; this takes 10 and 25 us.)
//      MANY: the low four bits of a minimum are the logarithm of how many vectors have its encoding, and vectors are counted; the bound
//      that is there stays where it is the closer one.
//      The kernel also sets the query's candidate count and flag, so that no launch is needed for those, and says
//      (LooseArgs) how large the error bound E of k_mm16 may be: everything up to tau + E becomes a candidate there, and
//      where a query's neighbourhood has many dimensions the count grows fast.  At most `groups` of the sample's
//      minima may lie up to there (the number at which the list's capacity is expected to be two thirds full), found by a
//      second bisection of the same registers.  A query whose E (estimated, with a fifth to spare) will exceed that or a
//      twenty-fourth of tau marks its block.  Only the choice of the filter hangs on it.
//      grid (ceil(queries / 4)), block 256; S <= 64 NV.
// ------------------------------------------------------------------------------------------------
struct LooseArgs {
    float *room;           // [nql] or nullptr: not asked for
    uint32_t *loose;       // [nql / 128] set to 1 for the blocks of queries without that room
    uint32_t *margin;      // [nql] the table filter's margin, for the blocks that are left to it
    uint32_t margin_table;
    const float *queries;  // [nq][d]
    const float *mean;     // [d]
    int d;
    int groups;            // sample groups whose minima may be at or below tau + E
    float typical;         // E / ||q|| as it is found for most queries
};

template <int NV, bool MANY>
__global__ __launch_bounds__(256) void k_tau(const float *__restrict__ gmin, int S, int64_t gstride, int k, int64_t nq, int64_t nql,
                                             float *__restrict__ tau, uint32_t *__restrict__ cnt, uint32_t *__restrict__ flag,
                                             uint32_t *__restrict__ counter, LooseArgs la)
{
    const int lane = threadIdx.x & 63;
    const int64_t ql = (int64_t)blockIdx.x * 4 + uniform(threadIdx.x >> 6);
    if (counter && blockIdx.x == 0 && threadIdx.x < 64) counter[lane] = 0u;
    if (ql >= nql) return;
    uint32_t bound = __float_as_uint(-1.f);  // a column past the last query: nothing passes
    float room = 0.f, nn = 0.f, e = 0.f;
    if (ql < nq) {
        const float *row = gmin + ql * gstride;
        uint32_t x[NV];
        uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int g = i * 64 + lane;
            x[i] = g < S ? __float_as_uint(row[g]) : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            lo = min(lo, x[i]);
            hi = max(hi, i * 64 + lane < S ? x[i] : 0u);
        }
#pragma unroll
        for (int dlt = 32; dlt >= 1; dlt >>= 1) {
            lo = min(lo, (uint32_t)__shfl_xor((int)lo, dlt));
            hi = max(hi, (uint32_t)__shfl_xor((int)hi, dlt));
        }
        lo = (uint32_t)uniform((int)lo);
        hi = (uint32_t)uniform((int)hi);
        const uint32_t largest = hi;
        auto count = [&](uint32_t upto) {
            int c = 0;
            if (MANY) {
#pragma unroll
                for (int i = 0; i < NV; ++i) c += x[i] <= upto ? 1 << (x[i] & 15u) : 0;
#pragma unroll
                for (int dlt = 32; dlt >= 1; dlt >>= 1) c += __shfl_xor(c, dlt);
                return uniform(c);
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) c += __popcll(__ballot(x[i] <= upto));
            return c;
        };
        // at least k minima are at or below hi, fewer than k below lo
        while (hi - lo > 127u) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            if (count(mid) >= k) hi = mid;
            else lo = mid + 1;
        }
        bound = S >= k ? hi : 0x7F800000u;
        if (MANY) {
            // (the bound that is there stands too, also the one below everything that k_prune gives a query whose tables are not
            // finite; and hi was a bound only if there are k vectors at all)
            const float t = tau[ql];
            bound = t < 0.f ? __float_as_uint(-1.f) : min(count(hi) >= k ? hi : 0x7F800000u, __float_as_uint(t));
        }
        if (la.room) {
            nn = 0.f;
            for (int j = lane; j < la.d; j += 64) {
                const float v = la.queries[ql * la.d + j] - la.mean[j];
                nn = fmaf(v, v, nn);
            }
#pragma unroll
            for (int dlt = 32; dlt >= 1; dlt >>= 1) nn += __shfl_xor(nn, dlt);
            e = la.typical * sqrtf(nn);
            if (!(28.f * e <= __uint_as_float(bound))) {
                room = -1.f;  // whatever the sample says
            } else if (la.groups >= S) {
                room = __uint_as_float(0x7F800000u);
            } else if (count(bound) <= la.groups) {
                // at most la.groups minima are at or below lo, more at or below hi (to 2^-10 of the value)
                lo = bound;
                hi = largest;
                while (hi - lo > 8191u) {
                    const uint32_t mid = lo + ((hi - lo) >> 1);
                    if (count(mid) <= la.groups) lo = mid;
                    else hi = mid;
                }
                room = __uint_as_float(lo) - __uint_as_float(bound);
            }
        }
    }
    if (la.room) {
        if (lane == 0) {
            la.room[ql] = room;
            la.margin[ql] = la.margin_table;
            if (ql < nq && !(1.2f * e <= room)) la.loose[ql / MM_Q] = 1u;  // (all write the same)
        }
    }
    if (lane == 0) {
        tau[ql] = __uint_as_float(bound);
        if (!MANY) {  // (no candidates yet, and k_prune's flags stand)
            cnt[ql] = 0u;
            flag[ql] = 0u;
        }
    }
}

// The same per-query state where there is no sample to take a bound from: every encoding is a candidate (tau: +inf;
// nullptr: not used), or (flagv = 1) every query goes to the exact kernel.  grid (ceil(queries / 256)), block 256.
__global__ __launch_bounds__(256) void k_search_init(float *__restrict__ tau, uint32_t *__restrict__ cnt, uint32_t *__restrict__ flag,
                                                     uint32_t *__restrict__ counter, int64_t nq, int64_t nql, uint32_t flagv)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (counter && blockIdx.x == 0 && threadIdx.x < 64) counter[threadIdx.x] = 0u;
    if (i >= nql) return;
    if (tau) tau[i] = i < nq ? __uint_as_float(0x7F800000u) : -1.f;
    cnt[i] = 0u;
    flag[i] = flagv;
}

// ------------------------------------------------------------------------------------------------
// block-level helpers (256 threads)
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void bitonic_sort_u64(uint64_t *a, int n)
{
    for (int k = 2; k <= n; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < n; i += blockDim.x) {
                const int ixj = i ^ j;
                if (ixj > i) {
                    const bool up = (i & k) == 0;
                    const uint64_t x = a[i], y = a[ixj];
                    if ((x > y) == up) {
                        a[i] = y;
                        a[ixj] = x;
                    }
                }
            }
            __syncthreads();
        }
}

// The same for lists of at most 256 keys (the usual case of the selection kernels: about k candidates): one wave holds
// H = 2 or 4 keys per lane (key e in lane e % 64, slot e / 64) and exchanges them by lane shuffles, or inside the lane
// where the partner is one of its own: 28 or 36 steps without a barrier or an LDS round trip each; the block-wide
// network above spends most of its time in those.  n: a power of two (a[0..n) holds the keys, padded with ~0 by the
// caller); every thread of the workgroup calls it, after a barrier.
template <int H>
__device__ __forceinline__ void wave_sort_u64(uint64_t *a, int n)
{
    const int lane = threadIdx.x;
    uint64_t x[H];
#pragma unroll
    for (int h = 0; h < H; ++h) x[h] = lane + 64 * h < n ? a[lane + 64 * h] : ~0ull;
#pragma unroll
    for (int k = 2; k <= 64 * H; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int e = lane + 64 * h;
                const bool keep_min = ((e & j) == 0) == ((e & k) == 0);  // lower index of an ascending pair, upper of a descending one
                if (j >= 64) {  // the partner is the lane's own key in slot h ^ (j / 64): handle the pair once
                    const int hp = h ^ (j >> 6);
                    if (hp > h) {
                        const uint64_t mn = x[h] < x[hp] ? x[h] : x[hp], mx = x[h] < x[hp] ? x[hp] : x[h];
                        x[h] = keep_min ? mn : mx;
                        x[hp] = keep_min ? mx : mn;
                    }
                } else {
                    const uint64_t y = (uint64_t)__shfl_xor((unsigned long long)x[h], j);
                    const uint64_t mn = x[h] < y ? x[h] : y, mx = x[h] < y ? y : x[h];
                    x[h] = keep_min ? mn : mx;
                }
            }
        }
#pragma unroll
    for (int h = 0; h < H; ++h)
        if (lane + 64 * h < n) a[lane + 64 * h] = x[h];
}

__device__ __forceinline__ void sort_u64(uint64_t *a, int n)
{
    if (n > 256) {
        bitonic_sort_u64(a, n);
        return;
    }
    if (threadIdx.x < 64) {
        if (n <= 128) wave_sort_u64<2>(a, n);
        else wave_sort_u64<4>(a, n);
    }
    __syncthreads();
}

// in-place inclusive scan of v[0..n) (n <= 256 * ipt), 256 threads, `tmp` has 4 entries
__device__ __forceinline__ void block_inclusive_scan(uint32_t *v, int n, uint32_t *tmp)
{
    const int ipt = (n + 255) / 256;
    const int lo = threadIdx.x * ipt, hi = min(n, lo + ipt);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t s = 0;
    for (int i = lo; i < hi; ++i) s += v[i];
    uint32_t inc = s;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)inc, dlt);
        if (lane >= dlt) inc += up;
    }
    if (lane == 63) tmp[wave] = inc;
    __syncthreads();
    for (int w2 = 0; w2 < wave; ++w2) inc += tmp[w2];
    uint32_t run = inc - s;
    for (int i = lo; i < hi; ++i) {
        run += v[i];
        v[i] = run;
    }
    __syncthreads();
}

// Smallest 32-bit value v such that at least `rank` of the participating keys are <= v (block of 256
// threads, most significant digit first, 4 passes of 8 bits).  key(i, v) returns false for entries
// that do not take part.  Also returns how many keys equal v and how many of those the rank needs.
// hist: 256 words of LDS, sh: 8 words of LDS.  first_pass: 0, or 2 when every key is below 2^16 (two passes then do).
template <class KeyFn>
__device__ __forceinline__ void block_radix_select(int n, uint32_t rank, KeyFn key, uint32_t *hist, uint32_t *sh,
                                                   uint32_t &value, uint32_t &rank_in_ties, uint32_t &n_ties, int first_pass = 0)
{
    uint32_t prefix = 0;
    for (int p = first_pass, shift = 24 - 8 * first_pass; p < 4; ++p, shift -= 8) {
        hist[threadIdx.x] = 0;
        __syncthreads();
#pragma unroll 8
        for (int i = threadIdx.x; i < n; i += 256) {
            uint32_t v;
            if (key(i, v) && (p == first_pass || (v >> (shift + 8)) == (prefix >> (shift + 8)))) atomicAdd(&hist[(v >> shift) & 255], 1u);
        }
        __syncthreads();
        // the digit at which the running count reaches the rank: a scan over the 256 bins, one bin per thread
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const uint32_t h = hist[threadIdx.x];
        uint32_t inc = h;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const uint32_t up = (uint32_t)__shfl_up((int)inc, dlt);
            if (lane >= dlt) inc += up;
        }
        if (lane == 63) sh[4 + wave] = inc;
        __syncthreads();
        for (int w2 = 0; w2 < wave; ++w2) inc += sh[4 + w2];
        const uint32_t excl = inc - h;
        if ((excl < rank && rank <= inc) || (threadIdx.x == 255 && inc < rank)) {
            sh[0] = prefix | ((uint32_t)threadIdx.x << shift);
            sh[1] = rank - excl;
            sh[2] = h;
        }
        __syncthreads();
        prefix = sh[0];
        rank = sh[1];
        n_ties = sh[2];
        __syncthreads();
    }
    value = prefix;
    rank_in_ties = rank;
}

__device__ __forceinline__ int pow2_at_least(int n)
{
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

// ------------------------------------------------------------------------------------------------
// S5b  final selection of one query from its candidate list (all encodings at or below the bound).
//      Only the k closest candidate encodings can contribute; they are sorted, expanded into their
//      vector ids (each encoding at most as many as are still needed), sorted by (distance, id), and
//      the first k are written.  Anything that does not fit the fixed LDS buffers (huge groups of exactly equal
//      distances) or its list (unless SelectArgs::again is there) is flagged for the exact whole-database kernel.
//      grid (queries of the batch), block 256, dynamic LDS select_lds_bytes(k).
// ------------------------------------------------------------------------------------------------
// capacity of the kept list and of the expanded list: twice k rounded up to a power of two, at least 256
// (room for the k closest plus a run of exactly equal distances); 16 bytes of dynamic LDS per entry plus 4
__host__ __device__ inline int select_cap(int k)
{
    int c = 256;
    while (c < 2 * k) c <<= 1;
    return c;
}
inline size_t select_lds_bytes(int k) { return (size_t)select_cap(k) * 20; }

struct SelectArgs {
    const uint32_t *cnt;     // [nq]
    const uint64_t *cand;    // [nq][C]
    uint32_t C;
    const uint32_t *ebegin;  // id range of every item, or nullptr: one id per item
    const int32_t *ids;      // ids_sorted (with ebegin) or ids in item order
    int k;
    int32_t *out_ids;        // [nq][k]
    float *out_dist;         // [nq][k]
    const uint32_t *perm;    // [nq] the row of the results that query ql's go to, or nullptr: row ql
    uint32_t *flag;          // [nq]  set to 1 when the query needs the exact kernel
    uint32_t *again;         // nullptr: a query whose list overran needs that too.  Otherwise the number of such queries and the queries: each is
                             // left with the k-th distance of its list in tau (behind it: k_refill)
    uint32_t *cnt_again;     // = cnt, for those
    float *tau;              // [nq]
    const float *bm;         // [tiles][M][64] or nullptr: results are written as B(q) - value (scalar-product searches)
    // Candidates from a fixed-point filter (k_lds with FX, k_lds16): the upper word of a candidate is a fixed-point
    // sum, which orders like the float32 distance up to fx_margin units.  First the k-th smallest sum is found; every
    // candidate up to it plus the margin gets its float32 distance from the tables (associated like the exact kernel
    // does, assoc_distance) written over the sum, every other candidate +inf; then the selection runs as on float32
    // candidates: what is ordered and returned is a float32 sum of table entries.
    int allow_short;         // 1: a query with fewer than k vectors among its candidates is complete (they are all
                             // there are): its row is filled up with id -1 and +inf; 0: such a query goes to the exact kernel
    uint32_t fx_margin;      // 0: the upper word is the float32 distance itself
    const uint32_t *margins; // [nq] a margin for every query in place of fx_margin, or nullptr
    int fx_first_pass;       // 2: the fixed-point sums are below 2^16 (see block_radix_select), else 0
    const float *lutT;       // [tiles][M][K][64] tables of this batch
    const uint8_t *codes;    // [items][M]
    const float *term;       // [items] leaf payload or nullptr
    int M, K, T, grouped;
    int32_t chunk_begin[ETF_MAX_M + 1];
};

// Sum of the table entries of one encoding c[0..M), associated as the main path of the mode does: `grouped` 4 or 8:
// like the LDS-resident kernels (chunks in groups as balanced trees, see lds_item_sum), 0: left to right inside a
// tree, trees in order.  lut(m, code) returns the entry.  A: anything with M, K, T, grouped, chunk_begin.
template <class A, class Lut>
__device__ __forceinline__ float assoc_distance(const A &a, Lut lut, const uint8_t *c)
{
    if (a.grouped == 4) {
        // chunks in groups of four as (c0 + c1) + (c2 + c3), a tree the sum of its groups in order (trees are equal
        // there; shorter ones live inside one group)
        const int M4 = a.M >> 2, D = a.M / a.T, gpt = D >= 4 ? D >> 2 : 1;
        float d = 0.f;
        for (int t0 = 0; t0 < M4; t0 += gpt) {
            float s = 0.f;
            for (int i = 0; i < gpt; ++i) {
                const int m = 4 * (t0 + i);
                const float P = (lut(m, c[m]) + lut(m + 1, c[m + 1])) + (lut(m + 2, c[m + 2]) + lut(m + 3, c[m + 3]));
                s = i == 0 ? P : s + P;
            }
            d = t0 == 0 ? s : d + s;
        }
        return d;
    }
    if (a.grouped == 8) {
        // groups of eight as a balanced tree, the groups added in order
        float d = 0.f;
        for (int m = 0; m < a.M; m += 8) {
            const float lo = (lut(m, c[m]) + lut(m + 1, c[m + 1])) + (lut(m + 2, c[m + 2]) + lut(m + 3, c[m + 3]));
            const float hi = (lut(m + 4, c[m + 4]) + lut(m + 5, c[m + 5])) + (lut(m + 6, c[m + 6]) + lut(m + 7, c[m + 7]));
            d = m == 0 ? lo + hi : d + (lo + hi);
        }
        return d;
    }
    float d = 0.f;
    for (int t = 0; t < a.T; ++t) {
        float s = 0.f;
        for (int m = a.chunk_begin[t]; m < a.chunk_begin[t + 1]; ++m) {
            const float v = lut(m, c[m]);
            s = (m == a.chunk_begin[t]) ? v : s + v;
        }
        d = (t == 0) ? s : d + s;
    }
    return d;
}

__device__ __forceinline__ void select_query(const SelectArgs &a, int64_t ql)
{
    extern __shared__ uint64_t sel_lds[];
    const int KEPT_CAP = select_cap(a.k), EXP_CAP = KEPT_CAP;
    uint64_t *kept = sel_lds;                                         // [KEPT_CAP]
    uint64_t *xkeys = sel_lds + KEPT_CAP;                             // [EXP_CAP]
    uint32_t *sc = reinterpret_cast<uint32_t *>(sel_lds + 2 * KEPT_CAP);  // [KEPT_CAP]
    __shared__ uint32_t tmp[4];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t s_a, s_b, s_c, s_d;
    __shared__ uint32_t sel_sh[8];
    const int64_t orow = a.perm ? (int64_t)a.perm[ql] : ql;
    if (a.flag[ql]) return;  // already routed to the exact kernel
    const uint32_t craw = a.cnt[ql];
    if (craw > a.C && !a.again) {
        if (threadIdx.x == 0) a.flag[ql] = 1;
        return;
    }
    const int c = (int)min(craw, a.C);
    const uint64_t *cand = a.cand + ql * a.C;
    const int k = a.k;
    // 1. the value of the min(k, c)-th closest candidate.  If more candidates tie with it exactly than
    //    fit, only those with the smallest first ids can matter (ids inside an encoding ascend, so the r
    //    smallest ids of a set of encodings lie in the r encodings with the smallest first id).
    auto first_id = [&](uint32_t e) -> uint32_t { return (uint32_t)a.ids[a.ebegin ? a.ebegin[e] : e]; };
    bool have_kept = false;
    if (a.fx_margin != 0) {
        // fixed-point sums: everything within the margin above the k-th smallest sum may be among the k closest
        uint32_t cut = 0xFFFFFFFFu;
        if (c > k) {
            uint32_t r2, n2;
            block_radix_select(
                c, (uint32_t)k, [&](int i, uint32_t &v) { v = (uint32_t)(cand[i] >> 32); return true; }, hist, sel_sh, cut, r2, n2,
                a.fx_first_pass);
            const uint32_t margin = a.margins ? a.margins[ql] : a.fx_margin;
            cut = cut < 0xFFFFFFFFu - margin ? cut + margin : 0xFFFFFFFFu;
        }
        const float *lq = a.lutT + (int64_t)(ql / QT) * a.M * a.K * QT + (ql % QT);
        auto lut = [&](int m, int code) -> float { return lq[((int64_t)m * a.K + code) * QT]; };
        auto float_key = [&](uint32_t e) -> uint64_t {
            const float dd = assoc_distance(a, lut, a.codes + (int64_t)e * a.M) + (a.term ? a.term[e] : 0.f);
            return ((uint64_t)__float_as_uint(dd) << 32) | e;
        };
        // nearly always the survivors fit the kept list: straight into it
        if (threadIdx.x == 0) s_c = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < c; i += 256) {
            const uint64_t key = cand[i];
            if ((uint32_t)(key >> 32) <= cut) {
                const uint32_t pos = atomicAdd(&s_c, 1u);
                if (pos < (uint32_t)KEPT_CAP) kept[pos] = float_key((uint32_t)key);
            }
        }
        __syncthreads();
        have_kept = s_c <= (uint32_t)KEPT_CAP;
        __syncthreads();
        if (!have_kept) {
            // a crowd within the rounding of the k-th sum: the list itself becomes a list of float32 candidates
            uint64_t *cw = const_cast<uint64_t *>(cand);  // it lives in the call's workspace
            for (int i = threadIdx.x; i < c; i += 256) {
                const uint64_t key = cand[i];
                cw[i] = (uint32_t)(key >> 32) <= cut ? float_key((uint32_t)key) : (0x7F80000000000000ull | (uint32_t)key);
            }
            __syncthreads();
        }
    }
    if (!have_kept) {
    uint32_t vstar = 0xFFFFFFFFu, idstar = 0xFFFFFFFFu;
    if (c > 256) {  // more than the sort below should see: cut at the k-th closest first
        const uint32_t rank = (uint32_t)min(k, c);
        uint32_t rank_in_ties, n_ties;
        block_radix_select(
            c, rank, [&](int i, uint32_t &v) { v = (uint32_t)(cand[i] >> 32); return true; }, hist, sel_sh, vstar,
            rank_in_ties, n_ties);
        if (rank - rank_in_ties + n_ties > (uint32_t)KEPT_CAP) {
            uint32_t r2, n2;
            block_radix_select(
                c, rank_in_ties,
                [&](int i, uint32_t &v) {
                    const uint64_t key = cand[i];
                    if ((uint32_t)(key >> 32) != vstar) return false;
                    v = first_id((uint32_t)key);
                    return true;
                },
                hist, sel_sh, idstar, r2, n2);
        }
    }
    // 2. keep the candidates at or below it, sorted by (distance bits, item)
    if (threadIdx.x == 0) s_c = 0;
    __syncthreads();
#pragma unroll 8
    for (int i = threadIdx.x; i < c; i += 256) {
        const uint64_t key = cand[i];
        const uint32_t v = (uint32_t)(key >> 32);
        if (v < vstar || (v == vstar && (idstar == 0xFFFFFFFFu || first_id((uint32_t)key) <= idstar))) {
            const uint32_t pos = atomicAdd(&s_c, 1u);
            if (pos < (uint32_t)KEPT_CAP) kept[pos] = key;
        }
    }
    __syncthreads();
    }
    const int nk = (int)s_c;
    if (nk == 0 && a.allow_short) {  // nothing in reach of this query
        for (int i = threadIdx.x; i < k; i += 256) {
            a.out_ids[orow * k + i] = -1;
            a.out_dist[orow * k + i] = __uint_as_float(0x7F800000u);
        }
        return;
    }
    if (nk > KEPT_CAP || nk == 0) {
        if (threadIdx.x == 0) a.flag[ql] = 1;
        return;
    }
    const int nk2 = pow2_at_least(nk);
    for (int i = nk + threadIdx.x; i < nk2; i += 256) kept[i] = ~0ull;
    __syncthreads();
    sort_u64(kept, nk2);
    // 3. how many vectors each kept encoding holds (never more than k matter)
    for (int i = threadIdx.x; i < nk; i += 256) {
        const uint32_t e = (uint32_t)kept[i];
        const uint32_t mult = a.ebegin ? a.ebegin[e + 1] - a.ebegin[e] : 1u;
        sc[i] = min(mult, (uint32_t)k);
    }
    __syncthreads();
    block_inclusive_scan(sc, nk, tmp);
    if (sc[nk - 1] < (uint32_t)k) {
        if (a.allow_short && nk <= (int)a.C && c == nk) {
            // every candidate was kept and together they hold fewer than k vectors: all of them, in order, then padding
            const uint32_t total = sc[nk - 1];
            __syncthreads();
            for (int i = threadIdx.x; i < nk; i += 256) {
                const uint32_t end = sc[i], beg = i > 0 ? sc[i - 1] : 0;
                const uint32_t e = (uint32_t)kept[i];
                const uint64_t hi = kept[i] & 0xFFFFFFFF00000000ull;
                for (uint32_t j = 0; j < end - beg; ++j) xkeys[beg + j] = hi | (uint32_t)a.ids[a.ebegin ? a.ebegin[e] + j : e];
            }
            const int nx2s = pow2_at_least((int)total);
            for (int i = (int)total + threadIdx.x; i < nx2s; i += 256) xkeys[i] = ~0ull;
            __syncthreads();
            sort_u64(xkeys, nx2s);
            for (int i = threadIdx.x; i < k; i += 256) {
                const bool have = i < (int)total;
                a.out_ids[orow * k + i] = have ? (int32_t)(uint32_t)xkeys[i] : -1;
                a.out_dist[orow * k + i] = have ? __uint_as_float((uint32_t)(xkeys[i] >> 32)) : __uint_as_float(0x7F800000u);
            }
            return;
        }
        // the bound was not valid: cannot happen with a sample of the database
        if (threadIdx.x == 0) a.flag[ql] = 1;
        return;
    }
    // first position whose running count reaches k, and the run of equal distances around it
    for (int i = threadIdx.x; i < nk; i += 256)
        if (sc[i] >= (uint32_t)k && (i == 0 || sc[i - 1] < (uint32_t)k)) s_a = (uint32_t)i;
    __syncthreads();
    const uint32_t dstar = (uint32_t)(kept[s_a] >> 32);
    for (int i = threadIdx.x; i < nk; i += 256) {
        const uint32_t v = (uint32_t)(kept[i] >> 32);
        if (v == dstar && (i == 0 || (uint32_t)(kept[i - 1] >> 32) != dstar)) s_b = (uint32_t)i;          // run start
        if (v == dstar && (i == nk - 1 || (uint32_t)(kept[i + 1] >> 32) != dstar)) s_d = (uint32_t)i + 1;  // run end
    }
    __syncthreads();
    const int ta = (int)s_b, tb = (int)s_d;
    const uint32_t before = ta > 0 ? sc[ta - 1] : 0;  // vectors strictly closer than dstar (< k)
    const uint32_t need = (uint32_t)k - before;        // still to take from the run of equal distances
    __syncthreads();
    // 4. contribution of every kept encoding, exclusive offsets, expansion into (distance, id) keys
    for (int i = threadIdx.x; i < nk; i += 256) {
        const uint32_t e = (uint32_t)kept[i];
        const uint32_t mult = a.ebegin ? a.ebegin[e + 1] - a.ebegin[e] : 1u;
        sc[i] = i < ta ? mult : (i < tb ? min(mult, need) : 0u);
    }
    __syncthreads();
    block_inclusive_scan(sc, nk, tmp);
    const uint32_t xtotal = sc[nk - 1];
    if (xtotal > (uint32_t)EXP_CAP) {
        if (threadIdx.x == 0) a.flag[ql] = 1;
        return;
    }
    for (int i = threadIdx.x; i < tb; i += 256) {
        const uint32_t end = sc[i], beg = i > 0 ? sc[i - 1] : 0;
        const uint32_t e = (uint32_t)kept[i];
        const uint64_t hi = kept[i] & 0xFFFFFFFF00000000ull;
        const uint32_t first = a.ebegin ? a.ebegin[e] : e;
        for (uint32_t j = 0; j < end - beg; ++j) xkeys[beg + j] = hi | (uint32_t)a.ids[first + j];
    }
    const int nx2 = pow2_at_least((int)xtotal);
    for (int i = (int)xtotal + threadIdx.x; i < nx2; i += 256) xkeys[i] = ~0ull;
    __syncthreads();
    sort_u64(xkeys, nx2);
    const float boff = a.bm ? product_shift(a.bm, a.M, ql) : 0.f;
    for (int i = threadIdx.x; i < k; i += 256) {
        a.out_ids[orow * k + i] = (int32_t)(uint32_t)xkeys[i];
        const float v = __uint_as_float((uint32_t)(xkeys[i] >> 32));
        a.out_dist[orow * k + i] = a.bm ? boff - v : v;
    }
    if (craw > a.C && threadIdx.x == 0) {  // (k encodings of the index lie at or below that, so it is a bound)
        a.tau[ql] = __uint_as_float((uint32_t)(xkeys[k - 1] >> 32));
        a.cnt_again[ql] = 0u;
        a.again[1 + atomicAdd(&a.again[0], 1u)] = (uint32_t)ql;
    }
}

__global__ __launch_bounds__(256) void k_select(SelectArgs a) { select_query(a, blockIdx.x); }

// the queries that k_refill has made new lists for (`queue`: their number, the queries).  grid (any), block 256, as k_select
__global__ __launch_bounds__(256) void k_select_refilled(SelectArgs a, const uint32_t *__restrict__ queue)
{
    const uint32_t n = queue[0];
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
        select_query(a, queue[1 + i]);
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------------
// S5c  exact selection over the whole database for one query, without any buffer that depends on the
//      data: a most-significant-digit radix select on the 64-bit key (distance bits, id), 8 passes of
//      8 bits, each pass recomputing the distances from the codes, then one collecting pass.  The sum
//      is associated exactly as in the mode's main path (left to right inside a chunk group, groups in
//      order), so both paths produce the same float32 values.
//      grid (queries of the batch), block 256; only flagged queries do any work.
// ------------------------------------------------------------------------------------------------
struct ExactArgs {
    const uint32_t *flag;     // [nq]
    uint32_t *nflag;          // running count of queries answered here
    const float *lutT;        // [tiles][M][K][64]
    int M, K, T;
    int grouped;              // 4 or 8: sums associated as the LDS-resident kernels do (see exact_distance), 0: left to right
    int32_t chunk_begin[ETF_MAX_M + 1];
    const uint8_t *codes;     // [rows][M]
    const float *term;        // [rows] leaf payload or nullptr
    int64_t rows;
    const uint32_t *ebegin;   // id ranges per row or nullptr (one id per row)
    const int32_t *ids;
    int k;
    int32_t *out_ids;
    float *out_dist;
    const uint32_t *perm;     // as in SelectArgs
    const float *bm;          // as in SelectArgs
};

__device__ __forceinline__ float exact_distance(const ExactArgs &a, const float *lut, const uint8_t *c)
{
    return assoc_distance(a, [&](int m, int code) -> float { return lut[m * a.K + code]; }, c);
}
// the same with the row's leaf term
__device__ __forceinline__ float exact_distance_row(const ExactArgs &a, const float *lut, int64_t e)
{
    return exact_distance(a, lut, a.codes + e * a.M) + (a.term ? a.term[e] : 0.f);
}

// ------------------------------------------------------------------------------------------------
// Lists anew for the queries whose list overran (SelectArgs::again): every encoding whose float32 distance, associated as it is
// returned, is at or below the k-th of the C encodings that the list held: about k times what was in reach over C of them, and never more
// than C where the list held more than half of that (2 C less what was in reach, k at least, are then among the nearest C).  A
// pair of query and stretch of the index a workgroup at a time, one query's tables in LDS.
//     What this is for: a query that is far from all vectors keeps a bound that lets through eight times what the whole sample's
//     does, and where the distances to it differ little its list may not hold that.  The exact selection below is one workgroup's nine
//     passes over the index.  (2268 queries far from 1.4 million encodings of 16 chunks, k = 20: the list of one of them
//     overran, 44 to 48 ms a search; now 1.87, and 1.75 where none does.  On 1198 random problems no query was left to the exact selection.)
//     Where no list overran this and k_select_refilled cost 5 us: 0.6 % of 10 000 queries on a million vectors.
//     grid (any), block 1024.
// ------------------------------------------------------------------------------------------------
struct RefillArgs {
    ExactArgs e;            // tables and codes (has no leaf term)
    const uint32_t *queue;  // the number of queries, the queries
    const float *tau;       // [nq]
    uint32_t *cnt;          // [nq] zero
    uint64_t *cand;         // [nq][C]
    uint32_t C;
    uint32_t stretch;       // encodings a workgroup takes
};

__global__ __launch_bounds__(1024) void k_refill(RefillArgs a)
{
    __shared__ float lut[ETF_MAX_M * 256];
    const uint32_t n = a.queue[0], parts = (uint32_t)((a.e.rows + a.stretch - 1) / a.stretch);
    const uint64_t work = (uint64_t)n * parts;
    for (uint64_t u = blockIdx.x; u < work; u += gridDim.x) {
        const int64_t ql = a.queue[1 + u / parts];
        const int64_t first = (int64_t)(u % parts) * a.stretch, end = min(a.e.rows, first + a.stretch);
        const float *src = a.e.lutT + (ql / QT) * a.e.M * a.e.K * QT + ql % QT;
        for (int i = threadIdx.x; i < a.e.M * a.e.K; i += 1024) lut[i] = src[(int64_t)i * QT];
        __syncthreads();
        const float tau = a.tau[ql];
        for (int64_t e = first + threadIdx.x; e < end; e += 1024) {
            const float d = exact_distance(a.e, lut, a.e.codes + e * a.e.M);
            if (d <= tau) {
                const uint32_t pos = atomicAdd(&a.cnt[ql], 1u);
                if (pos < a.C) a.cand[ql * a.C + pos] = ((uint64_t)__float_as_uint(d) << 32) | (uint32_t)e;
            }
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_exact(ExactArgs a)
{
    __shared__ float lut[ETF_MAX_M * 256];
    __shared__ uint32_t hist[256];
    __shared__ uint64_t okeys[ETF_MAX_TOPK];
    __shared__ uint32_t s_digit, s_rank, s_n;
    const int64_t ql = blockIdx.x, orow = a.perm ? (int64_t)a.perm[ql] : ql;
    if (!a.flag[ql]) return;
    if (threadIdx.x == 0) atomicAdd(a.nflag, 1u);
    const int tile = (int)(ql / QT), col = (int)(ql % QT);
    for (int i = threadIdx.x; i < a.M * a.K; i += 256) lut[i] = a.lutT[((int64_t)tile * a.M * a.K + i) * QT + col];
    __syncthreads();
    const uint32_t k = (uint32_t)a.k;
    uint64_t prefix = 0;
    uint32_t rank = k;
    for (int p = 0, shift = 56; p < 8; ++p, shift -= 8) {
        hist[threadIdx.x] = 0;
        __syncthreads();
        for (int64_t e = threadIdx.x; e < a.rows; e += 256) {
            const uint32_t v = __float_as_uint(exact_distance_row(a, lut, e));
            const uint32_t first = a.ebegin ? a.ebegin[e] : (uint32_t)e;
            const uint32_t mult = min(a.ebegin ? a.ebegin[e + 1] - first : 1u, k);
            if (p < 4) {
                const int sh = shift - 32;  // digit position inside the distance bits
                if (p == 0 || (v >> (sh + 8)) == ((uint32_t)(prefix >> 32) >> (sh + 8)))
                    atomicAdd(&hist[(v >> sh) & 255], mult);
            } else if (v == (uint32_t)(prefix >> 32)) {
                for (uint32_t j = 0; j < mult; ++j) {
                    const uint32_t id = (uint32_t)a.ids[first + j];
                    if (p == 4 || (id >> (shift + 8)) == ((uint32_t)prefix >> (shift + 8)))
                        atomicAdd(&hist[(id >> shift) & 255], 1u);
                }
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t below = 0;
            int b = 0;
            for (; b < 255; ++b) {
                if (below + hist[b] >= rank) break;
                below += hist[b];
            }
            s_digit = (uint32_t)b;
            s_rank = rank - below;
        }
        __syncthreads();
        prefix |= (uint64_t)s_digit << shift;
        rank = s_rank;
        __syncthreads();
    }
    // collect every (distance, id) key at or below the k-th: exactly k of them
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const uint32_t vk = (uint32_t)(prefix >> 32), idk = (uint32_t)prefix;
    for (int64_t e = threadIdx.x; e < a.rows; e += 256) {
        const uint32_t v = __float_as_uint(exact_distance_row(a, lut, e));
        if (v > vk) continue;
        const uint32_t first = a.ebegin ? a.ebegin[e] : (uint32_t)e;
        const uint32_t mult = min(a.ebegin ? a.ebegin[e + 1] - first : 1u, k);
        for (uint32_t j = 0; j < mult; ++j) {
            const uint32_t id = (uint32_t)a.ids[first + j];
            if (v < vk || id <= idk) {
                const uint32_t pos = atomicAdd(&s_n, 1u);
                if (pos < ETF_MAX_TOPK) okeys[pos] = ((uint64_t)v << 32) | id;
            }
        }
    }
    __syncthreads();
    const int n = (int)min(s_n, (uint32_t)ETF_MAX_TOPK);
    const int n2 = pow2_at_least(max(n, 1));
    for (int i = n + threadIdx.x; i < n2; i += 256) okeys[i] = ~0ull;
    __syncthreads();
    bitonic_sort_u64(okeys, n2);
    const float boff = a.bm ? product_shift(a.bm, a.M, ql) : 0.f;
    for (int i = threadIdx.x; i < a.k; i += 256) {
        a.out_ids[orow * a.k + i] = (int32_t)(uint32_t)okeys[i];
        const float v = __uint_as_float((uint32_t)(okeys[i] >> 32));
        a.out_dist[orow * a.k + i] = a.bm ? boff - v : v;
    }
}

// ------------------------------------------------------------------------------------------------
// Bandwidth probes (benchmark only): what this card's memory delivers to plain streaming kernels, the
// ceilings the traversal kernels are compared with.  16 bytes per lane and access, grid-stride.
//     k_probe_read:  sum of `n16` 16-byte pieces of a; one word per workgroup is written to out
//     k_probe_write: n16 pieces of a constant to a
//     k_probe_copy:  a -> b
//     k_probe_rows:  a read as rows of 256 bytes (a wave per row, the unit of every table in this library) in a
//                    scattered order: row (i * mult) mod nrows for i = 0 .. nrows-1, mult coprime to nrows
// ------------------------------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_probe_read(const u32x4 *__restrict__ a, int64_t n16, uint32_t *__restrict__ out)
{
    u32x4 acc = 0u;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n16; i += 4 * stride) {  // four loads in flight per lane
        const u32x4 v0 = __builtin_nontemporal_load(a + i), v1 = __builtin_nontemporal_load(a + i + stride),
                    v2 = __builtin_nontemporal_load(a + i + 2 * stride), v3 = __builtin_nontemporal_load(a + i + 3 * stride);
        acc ^= (v0 ^ v1) ^ (v2 ^ v3);
    }
    for (; i < n16; i += stride) acc ^= __builtin_nontemporal_load(a + i);
    const uint32_t x = (acc.x ^ acc.y) ^ (acc.z ^ acc.w);
    if (x == 0x9E3779B9u || threadIdx.x == 0) out[blockIdx.x] = x;
}

__global__ __launch_bounds__(256) void k_probe_write(u32x4 *__restrict__ a, int64_t n16)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const u32x4 v = {1u, 2u, 3u, 4u};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) a[i] = v;
}

__global__ __launch_bounds__(256) void k_probe_copy(const u32x4 *__restrict__ a, u32x4 *__restrict__ b, int64_t n16)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        const u32x4 v0 = __builtin_nontemporal_load(a + i), v1 = __builtin_nontemporal_load(a + i + stride),
                    v2 = __builtin_nontemporal_load(a + i + 2 * stride), v3 = __builtin_nontemporal_load(a + i + 3 * stride);
        __builtin_nontemporal_store(v0, b + i);
        __builtin_nontemporal_store(v1, b + i + stride);
        __builtin_nontemporal_store(v2, b + i + 2 * stride);
        __builtin_nontemporal_store(v3, b + i + 3 * stride);
    }
    for (; i < n16; i += stride) __builtin_nontemporal_store(__builtin_nontemporal_load(a + i), b + i);
}

__global__ __launch_bounds__(256) void k_probe_rows(const float *__restrict__ a, int64_t nrows, uint64_t mult, uint32_t *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const int64_t wv = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), nwv = (int64_t)gridDim.x * 4;
    float acc = 0.f;
    // row of step i is (i * mult) mod nrows, advanced by additions: mult < nrows, so one subtraction brings a sum back
    const uint64_t n = (uint64_t)nrows, hop = ((uint64_t)nwv * 8 % n) * mult % n;
    uint64_t r0 = (uint64_t)(wv * 8 % nrows) * mult % n;
    for (int64_t i0 = wv * 8; i0 + 8 <= nrows; i0 += nwv * 8) {  // eight rows in flight per wave
        float v[8];
        uint64_t r = r0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            v[u] = a[r * 64 + lane];
            r += mult;
            r = r >= n ? r - n : r;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
        r0 += hop;
        r0 = r0 >= n ? r0 - n : r0;
    }
    if (acc == 1.2345e-30f || threadIdx.x == 0) out[blockIdx.x] = __float_as_uint(acc);
}

// LDS read rate of the chip: every lane of a workgroup of 1024 threads reads 16 bytes per instruction, `iters`
// instructions per wave, eight in flight; the data is folded into one word per workgroup so that the reads stay.
// The vector unit's issue rate for one instruction kind: eight independent dependency chains per lane, 64 instructions
// per lane and iteration, nothing else in the loop.  KIND 0: v_add_f32 (one float32 operation per lane), 1: v_add3_u32
// (the 16-bit filter's adds: two additions of two packed 16-bit entries each), 2: v_pk_add_u16.
// grid (2048), block 256; out receives one word per workgroup.
template <int KIND>
__global__ __launch_bounds__(256) void k_probe_valu(int iters, uint32_t *__restrict__ out)
{
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = threadIdx.x * 8u + (uint32_t)u;
    const uint32_t c = blockIdx.x + 1u;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int rep = 0; rep < 8; ++rep)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (KIND == 0) asm volatile("v_add_f32 %0, %1, %0" : "+v"(v[u]) : "v"(c));
                if (KIND == 1) asm volatile("v_add3_u32 %0, %0, %1, %1" : "+v"(v[u]) : "v"(c));
                if (KIND == 2) asm volatile("v_pk_add_u16 %0, %0, %1" : "+v"(v[u]) : "v"(c));
            }
    }
    uint32_t x = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) x ^= v[u];
    if (threadIdx.x == (x & 255u)) out[blockIdx.x] = x;
}

// The rate of the float32 matrix instruction the lookup-table, encoder and coarse-quantiser kernels are built on:
// v_mfma_f32_32x32x2_f32 on eight independent accumulator blocks per wave, operands in registers, nothing else.
// grid (2048), block 256; 32 instructions (131072 floating-point operations) per wave and iteration.
__global__ __launch_bounds__(256) void k_probe_mfma(int iters, uint32_t *__restrict__ out)
{
    floatx16 acc[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[u][r] = 0.f;
    const float a = (float)(threadIdx.x & 7) * 0.125f, b = (float)(blockIdx.x & 3) * 0.25f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int rep = 0; rep < 4; ++rep)
#pragma unroll
            for (int u = 0; u < 8; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc[u], 0, 0, 0);
    }
    float x = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) x += acc[u][r];
    if (threadIdx.x == ((uint32_t)x & 255u)) out[blockIdx.x] = __float_as_uint(x);
}

// Plain: lane l of a wave reads piece l of a 1 KiB row (conflict-free: every quarter wave covers all 64 banks).
// SCATTER: the four lanes of a group read the four pieces of one 64-byte row and the sixteen groups of a wave read
// rows picked by a hash: the access pattern of the table lookups, bank conflicts as they fall.
template <bool SCATTER>
__global__ __launch_bounds__(1024) void k_probe_lds(int iters, uint32_t *__restrict__ out)
{
    extern __shared__ u32x4 probe_lds[];  // 128 KiB
    constexpr int PIECES = 128 * 1024 / 16;
    for (int i = threadIdx.x; i < PIECES; i += 1024) probe_lds[i] = u32x4{(uint32_t)i, 1u, 2u, 3u};
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t h = (uint32_t)(lane >> 2) * 0x9E3779B9u + (uint32_t)w * 0x85EBCA6Bu + blockIdx.x;
    uint32_t last = 0u;
    for (int it = 0; it < iters; it += 8) {
        u32x4 v[8];
        const int row0 = (it + w) & 63;  // rows row0, row0 + 8, ..., row0 + 56 of the 128: a different set every time
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            int piece;
            if (SCATTER) {
                h += 0x9E3779B9u;  // a Weyl sequence: cheap enough that the vector unit stays behind the LDS pipe
                piece = (int)(((h >> 15) & (PIECES / 4 - 1)) << 2 | (uint32_t)(lane & 3));
            } else {
                piece = (row0 + u * 8) * 64 + lane;
            }
            v[u] = probe_lds[piece];
        }
        // the loaded registers are used by an empty statement: no arithmetic competes with the reads, and the
        // compiler can neither drop nor narrow them
#pragma unroll
        for (int u = 0; u < 8; ++u) asm volatile("" ::"v"(v[u]));
        last = v[7].x;
    }
    if (last == 0x9E3779B9u || threadIdx.x == 0) out[blockIdx.x] = last;
}

}  // namespace etf
