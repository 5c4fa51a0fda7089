// Which parts of the index a group of queries can do without (included by etf_device.hip behind etf_kernels.hip.h).
//
//     Queries that are near each other need the same few parts of a clustered database.  So the queries of a large batch are
//     put in the order of their nearest codewords of the first two chunks before their tables are built (k_order_keys,
//     k_order_sort, k_order_gather; of the kernels behind them only those that write a query's results know of it: k_select, k_refill's
//     second selection and k_exact).  The index is taken in blocks of 64 encodings (or 2, 4, .. times that), which are ranges of the
//     tree's leaves.  For every sub-tile of the 16-bit filter k_prune makes a table for each of the first three chunks: how much of what
//     a query's bound leaves above its least sum an entry takes, least over the sub-tile's queries.  A block is kept if a prefix of
//     three chunks in its range can stay within 1.  k_lds16<.., WALK_NEAR> takes a closer bound from the nearest of the kept blocks,
//     k_prune goes over all blocks again with that, and k_lds16<.., WALK_KEPT> walks the blocks that are then kept.
//     Nothing at or below a bound is lost: a float32 sum of at most 16 entries moves by less than 16 2^-24 of itself with the
//     order of its additions, and the bound is widened by 2^-16 of itself.
//     Measured (MI355X), 10^6 x 128 in 8 chunks, 64 overlapping clusters, 10 000 queries, k = 100: the filter pass 1.31 -> 0.40 ms (a fifth
//     of the blocks kept, 220 candidates a query in place of 900), the bound's sample 0.33 -> 0.20 (the first 0.08, the near walk
//     0.12), k_select 0.165 -> 0.13, against 0.03 for the queries' order, 0.05 and 0.03 for k_prune, 0.03 for the second k_tau and
//     0.01 for k_units: 1.87 -> 0.93 ms.  10^7 x 128 in 16 chunks, 1024 clusters: 14.9 -> 4.1 to 4.4.
#pragma once

namespace etf {

// ------------------------------------------------------------------------------------------------
// The nearest codeword of every query in the chunk that the index has at position blockIdx.y (0 or 1), as plain float32 sums:
// only the order of the queries comes from it.  A wave holds 16 codewords, a lane a query; the codewords come through the scalar cache.
//     keys[2][nql].  grid (tiles, 2), block 1024.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_order_keys(const float *__restrict__ queries, int64_t nq, int64_t nql, int d, int ds, int K,
                                                     const float *__restrict__ cb, ChunkOrder ord, uint8_t *__restrict__ keys)
{
    __shared__ float s_best[16][64];
    __shared__ uint8_t s_code[16][64];
    const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
    const int ms = ord.src[blockIdx.y];
    const int64_t q = (int64_t)blockIdx.x * QT + lane;
    const float *row = queries + (q < nq ? q : 0) * d + (int64_t)ms * ds;
    const float *cw = cb + (int64_t)ms * K * ds;
    int at[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) at[c] = min(w * 16 + c, K - 1) * ds;
    float acc[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) acc[c] = 0.f;
    // (pieces of four dimensions; of chunks of 64 dimensions and more every so many-th piece, eight to fifteen in all, which orders the
    // queries as well)
    const int step = 4 * max(1, ds / 32);
    int j = 0;
    for (; j + 4 <= ds; j += step) {
        const float x0 = row[j], x1 = row[j + 1], x2 = row[j + 2], x3 = row[j + 3];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const float *p = cw + at[c] + j;
            const float a = x0 - p[0], b = x1 - p[1], e = x2 - p[2], f = x3 - p[3];
            acc[c] = fmaf(f, f, fmaf(e, e, fmaf(b, b, fmaf(a, a, acc[c]))));
        }
    }
    for (j = ds < 32 ? ds & ~3 : ds; j < ds; ++j) {
        const float x = row[j];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const float a = x - cw[at[c] + j];
            acc[c] = fmaf(a, a, acc[c]);
        }
    }
    float best = acc[0];
    int code = min(w * 16, K - 1);
#pragma unroll
    for (int c = 1; c < 16; ++c)
        if (acc[c] < best) {
            best = acc[c];
            code = min(w * 16 + c, K - 1);
        }
    s_best[w][lane] = best;
    s_code[w][lane] = (uint8_t)code;
    __syncthreads();
    if (w != 0) return;
#pragma unroll
    for (int i = 1; i < 16; ++i)
        if (s_best[i][lane] < best) {
            best = s_best[i][lane];
            code = s_code[i][lane];
        }
    keys[(int64_t)blockIdx.y * nql + q] = (uint8_t)code;
}

// ------------------------------------------------------------------------------------------------
// Positions of the queries in the order of (codeword of chunk 0, codeword of chunk 1 mod 16): a counting sort by one workgroup
// (4096 counts in LDS; queries of one codeword of chunk 1 stay together, and what a codeword of chunk 0 has, a few sub-tiles,
// needs no finer division).  Inside a bin the order is whichever comes first; results do not depend on it.
//     perm[position] = query.  Clears `words` of state and the number of queries whose lists overran.  grid 1, block 1024.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_order_sort(const uint8_t *__restrict__ keys, int64_t nq, int64_t nql, uint32_t *__restrict__ perm,
                                                     uint32_t *__restrict__ state, int words, uint32_t *__restrict__ again)
{
    __shared__ uint32_t bin[4096];
    __shared__ uint32_t wsum[16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int i = t; i < words; i += 1024) state[i] = 0u;
    if (t == 0) again[0] = 0u;
    for (int i = t; i < 4096; i += 1024) bin[i] = 0u;
    __syncthreads();
    auto bin_of = [&](int64_t q) { return ((uint32_t)keys[q] << 4) | (keys[nql + q] & 15u); };
    uint32_t held[16];  // the bins of the first 16 x 1024 queries
#pragma unroll
    for (int i = 0; i < 16; ++i) held[i] = t + i * 1024 < nq ? bin_of(t + i * 1024) : 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (t + i * 1024 < nq) atomicAdd(&bin[held[i]], 1u);
    for (int64_t q = t + 16 * 1024; q < nq; q += 1024) atomicAdd(&bin[bin_of(q)], 1u);
    __syncthreads();
    uint32_t v[4], sum = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = bin[4 * t + i];
        sum += v[i];
    }
    uint32_t upto = sum;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)upto, dlt);
        if (lane >= dlt) upto += o;
    }
    if (lane == 63) wsum[w] = upto;
    __syncthreads();
    uint32_t before = upto - sum;
    for (int i = 0; i < w; ++i) before += wsum[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        bin[4 * t + i] = before;
        before += v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (t + i * 1024 < nq) perm[atomicAdd(&bin[held[i]], 1u)] = (uint32_t)(t + i * 1024);
    for (int64_t q = t + 16 * 1024; q < nq; q += 1024) perm[atomicAdd(&bin[bin_of(q)], 1u)] = (uint32_t)q;
}

// ------------------------------------------------------------------------------------------------
// The queries in their new order (a wave per query), and the first three chunks of the first and the last encoding of every
// block of 2^shift x 64.  grid (ceil(nq / 4) + ceil(nblk / 256)), block 256.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_order_gather(const float *__restrict__ queries, int64_t nq, int d, const uint32_t *__restrict__ perm,
                                                      float *__restrict__ sorted, const uint8_t *__restrict__ ecodes, int64_t nitems, int M,
                                                      int shift, int nblk, uint2 *__restrict__ span)
{
    const int64_t rows = (nq + 3) / 4;
    if ((int64_t)blockIdx.x >= rows) {
        const int64_t b = ((int64_t)blockIdx.x - rows) * 256 + threadIdx.x;
        if (b >= nblk) return;
        const int64_t first = b << (6 + shift), last = min(nitems, (b + 1) << (6 + shift)) - 1;
        const uint8_t *f = ecodes + first * M, *l = ecodes + last * M;
        span[b] = make_uint2(((uint32_t)f[0] << 16) | ((uint32_t)f[1] << 8) | f[2], ((uint32_t)l[0] << 16) | ((uint32_t)l[1] << 8) | l[2]);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int64_t pos = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (pos >= nq) return;
    const float *src = queries + (int64_t)perm[pos] * d;
    float *dst = sorted + pos * d;
    for (int j = lane; j < d; j += 64) dst[j] = src[j];
}

// ------------------------------------------------------------------------------------------------
// The blocks that a sub-tile of Qs queries needs.  Let s be a query's bound less its least entry of every chunk, e_m(c) the
// excess of an entry of chunk m over the chunk's least.  An encoding can matter to the query only where the sum of its excesses is
// at most s, and to any query of the sub-tile only where the sum of x_m(c_m) is at most 1, with x the least e / s among its queries:
// a table of 256 numbers for every chunk, whatever the number of nodes.  (For queries in order that keeps hardly more than a test of every
// query at every node does: of 64 overlapping clusters 17.2 % either way, of 1024 45.2 % in place of 45.0.)  A block is a
// range of the tree's leaves: the least sum of the first three chunks in its range comes from tables of range minima.  The nearest
// `near_blocks` by that sum are what k_lds16<.., WALK_NEAR> takes a closer bound from: the sums in 255 classes, all of the
// blocks of the classes that fit and of the next class every so many-th.
//     again: with the closer bound, all kept blocks in any order; the least entries are there from the first call.
//     Bound by the read of the sub-tile's tables (10 000 queries, 8 chunks of 700 000 encodings: 50 us; 16 chunks of 6.5 million: 172), again
//     by the chain of its steps (30 and 101 us).  grid (sub-tiles that hold a query), block 1024.
// ------------------------------------------------------------------------------------------------
struct PruneArgs {
    const float *lutT;     // [tiles][M][K][64]
    float *tau;            // [tiles*64]
    uint32_t *flag;        // [tiles*64] set to 1 for the exact kernel
    float *least;          // [4][tiles*64] the sum of a query's least entries, those of the first three chunks
    int64_t nql;           // tiles*64
    const uint2 *span;     // [nblk]
    int nblk;              // blocks of the index, at most 2^16
    int M, K;
    int64_t nq;
    int near_blocks;
    uint8_t *kind;         // [sub-tiles][nblk] classes
    uint16_t *list;        // [sub-tiles][nblk] the nearest blocks, or all that are kept
    uint32_t *count;       // [sub-tiles] how many are kept (again)
    uint4 *near;           // [sub-tiles] blocks of the list to take all of, the number of those to take some of, how many of them
    uint32_t *state;       // per block of MM_Q queries: kept blocks, sub-tiles counted (high byte)
    uint32_t *loose;       // per block of MM_Q queries: set where k_mm16 is to leave it, or nullptr: it does not run
    float mm_share;        // ... which is where less than this share of the index is kept
    bool again;
};
constexpr int PRUNE_BLOCKS = 1 << 16;  // (a list's entries have 16 bits, the sum of eight sub-tiles' kept blocks 24)

template <int Qs>
__global__ __launch_bounds__(1024) void k_prune(PruneArgs a)
{
    __shared__ uint32_t least[ETF_MAX_M][Qs];   // bits
    __shared__ float inv[Qs], low[3][Qs];       // 1 / s, the least entries of the first three chunks
    __shared__ float x[3][8][256];              // [m][l][c]: the least x_m of 2^l codewords from c on
    __shared__ uint32_t hist[256];
    __shared__ uint32_t part[4];                // where the next block of the list's two parts goes; the class of the second
    __shared__ uint32_t endless, narrowest;     // an infinite bound; the least s (bits)
    constexpr int P = Qs / 4;                   // 16-byte pieces of a row
    const float inf = __uint_as_float(0x7F800000u);
    const int s = blockIdx.x, tile = s / (QT / Qs), sub = s % (QT / Qs);
    const int t = threadIdx.x, lane = t & 63, w = uniform(t >> 6);
    const int M = a.M, K = a.K;
    const int64_t col = (int64_t)tile * QT + sub * Qs;
    if (t < 256) hist[t] = 0u;
    if (t == 0) {
        endless = 0u;
        narrowest = 0x7F800000u;
    }
    if (t < 4) part[t] = 0u;
    const float *src = a.lutT + (int64_t)tile * M * K * QT + sub * Qs;
    if (!a.again) {
        for (int i = t; i < M * Qs; i += 1024) (&least[0][0])[i] = 0x7F800000u;
        __syncthreads();
        const int p = t % P, r0 = t / P;
        constexpr int RS = 1024 / P, R = 256 / RS;  // rows between a thread's, and how many it has of a chunk
        for (int m0 = 0; m0 < M; m0 += 4) {         // (M is 8 or 16)
            float4 e[4][R];
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    e[m][r] = *reinterpret_cast<const float4 *>(src + ((int64_t)(m0 + m) * K + min(r0 + r * RS, K - 1)) * QT + p * 4);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                float lo[4] = {inf, inf, inf, inf};
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    lo[0] = fminf(lo[0], e[m][r].x);
                    lo[1] = fminf(lo[1], e[m][r].y);
                    lo[2] = fminf(lo[2], e[m][r].z);
                    lo[3] = fminf(lo[3], e[m][r].w);
                }
                // (table entries are not negative: their bits order like they do)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    uint32_t x = __float_as_uint(lo[v]);
#pragma unroll
                    for (int dlt = 32; dlt >= P; dlt >>= 1) x = min(x, (uint32_t)__shfl_xor((int)x, dlt));
                    if (lane < P) atomicMin(&least[m0 + m][p * 4 + v], x);
                }
            }
        }
    }
    __syncthreads();
    if (t < Qs) {
        float tau = a.tau[col + t];
        float sum = 0.f;
        if (a.again) {
            sum = a.least[col + t];
#pragma unroll
            for (int m = 0; m < 3; ++m) low[m][t] = a.least[(m + 1) * a.nql + col + t];
        } else {
            for (int m = 0; m < M; ++m) sum += __uint_as_float(least[m][t]);
            a.least[col + t] = sum;
#pragma unroll
            for (int m = 0; m < 3; ++m) a.least[(m + 1) * a.nql + col + t] = low[m][t] = __uint_as_float(least[m][t]);
        }
        // A query without a finite entry in some chunk (a NaN or an infinity in it, or its squares are infinite) has no finite distance:
        // the exact selection answers it, and a bound below everything keeps it from keeping all of the index for its sub-tile.
        if (!a.again && tau >= 0.f && sum == inf) {
            tau = a.tau[col + t] = -1.f;
            a.flag[col + t] = 1u;
            if (a.loose) a.loose[(col + t) / MM_Q] = 1u;  // (k_mm16 scales a block by its queries: not for it)
        }
        if (tau == inf) endless = 1u;  // (fewer than k finite distances in the sample: everything is kept)
        // a column past the last query has a negative bound too: inv < 0, nothing matters
        float room = tau >= 0.f ? fmaxf(fmaf(tau, 1.52587890625e-5f, tau) - sum, 1e-30f) : -1.f;
        if (!a.again) {
            // Nearness goes by the geometric mean of the query's s and the least one: where a cluster has fewer encodings than the
            // sample needs, a bound reaches to the next cluster, twenty times too far, and the query's neighbours would be all there is.
            if (room >= 0.f) atomicMin(&narrowest, __float_as_uint(room));
            __builtin_amdgcn_wave_barrier();
            if (room >= 0.f) room = sqrtf(room) * sqrtf(__uint_as_float(narrowest));
        }
        inv[t] = room >= 0.f ? 1.f / room : -1.f;
    }
    __syncthreads();
    const int xm = t >> 8, xc = t & 255;  // a thread a codeword
    if (xm < 3) {
        const float *row = src + ((int64_t)xm * K + min(xc, K - 1)) * QT;
        float4 e[Qs / 4];
#pragma unroll
        for (int i = 0; i < Qs / 4; ++i) e[i] = *reinterpret_cast<const float4 *>(row + 4 * i);
        float v = inf;
#pragma unroll
        for (int i = 0; i < Qs / 4; ++i) {
            const float u[4] = {e[i].x, e[i].y, e[i].z, e[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float g = inv[4 * i + j];
                if (g >= 0.f) v = fminf(v, (u[j] - low[xm][4 * i + j]) * g);
            }
        }
        x[xm][0][xc] = endless != 0u ? 0.f : xc < K ? v : inf;
    }
    for (int l = 1; l < 8; ++l) {
        __syncthreads();
        if (xm < 3) x[xm][l][xc] = fminf(x[xm][l - 1][xc], x[xm][l - 1][min(xc + (1 << (l - 1)), 255)]);
    }
    __syncthreads();
    auto least_of = [&](int m, int from, int to) -> float {  // of codewords from .. to
        if (from > to) return inf;
        const int l = min(31 - __builtin_clz(to - from + 1), 7);
        return fminf(x[m][l][from], x[m][l][to + 1 - (1 << l)]);  // (256 codewords: twice 128)
    };
    // the class of a block, 255: not kept.  It goes by the least sum in its range of prefixes
    auto class_of = [&](uint2 r) -> uint32_t {
        const int a0 = (int)(r.x >> 16), a1 = (int)((r.x >> 8) & 255u), a2 = (int)(r.x & 255u);
        const int b0 = (int)(r.y >> 16), b1 = (int)((r.y >> 8) & 255u), b2 = (int)(r.y & 255u);
        float f;
        if (a0 != b0) f = fminf(fminf(x[0][0][a0] + least_of(1, a1, 255), x[0][0][b0] + least_of(1, 0, b1)), least_of(0, a0 + 1, b0 - 1));
        else if (a1 != b1)
            f = x[0][0][a0] + fminf(fminf(x[1][0][a1] + least_of(2, a2, 255), x[1][0][b1] + least_of(2, 0, b2)), least_of(1, a1 + 1, b1 - 1));
        else f = x[0][0][a0] + x[1][0][a1] + least_of(2, a2, b2);
        return f <= 1.f ? min((uint32_t)(255.f * __builtin_amdgcn_sqrtf(f)), 254u) : 255u;
    };
    // eight blocks of a thread at a time: a wave has 64 neighbours of each
    constexpr int AT = 8;
    uint16_t *list = a.list + (int64_t)s * a.nblk;
    if (a.again) {
        // all that are kept
        for (int i0 = 0; i0 < a.nblk; i0 += AT * 1024) {
            uint2 r[AT];
            uint64_t g[AT];
            uint32_t n = 0u, at = 0u;
#pragma unroll
            for (int u = 0; u < AT; ++u) r[u] = a.span[min(i0 + u * 1024 + t, a.nblk - 1)];
#pragma unroll
            for (int u = 0; u < AT; ++u) {
                g[u] = __ballot(i0 + u * 1024 + t < a.nblk && class_of(r[u]) != 255u);
                n += (uint32_t)__popcll(g[u]);
            }
            if (n == 0u) continue;
            if (lane == 0) at = atomicAdd(&part[0], n);
            at = (uint32_t)uniform((int)at);
#pragma unroll
            for (int u = 0; u < AT; ++u) {
                if ((g[u] >> lane) & 1ull)
                    list[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(g[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)g[u], 0u))] = (uint16_t)(i0 + u * 1024 + t);
                at += (uint32_t)__popcll(g[u]);
            }
        }
        __syncthreads();
        if (t == 0) {
            const uint32_t n = part[0];
            a.count[s] = n;
            if (a.loose) {
                const int b = s / (MM_Q / Qs);
                const uint32_t subs = (uint32_t)((min<int64_t>(MM_Q, a.nq - (int64_t)b * MM_Q) + Qs - 1) / Qs);
                const uint32_t was = atomicAdd(&a.state[b], n | (1u << 24));
                if ((was >> 24) + 1u == subs && (float)((was & 0xFFFFFFu) + n) < a.mm_share * (float)a.nblk * (float)subs) a.loose[b] = 1u;
            }
        }
        return;
    }
    uint8_t *kind = a.kind + (int64_t)s * a.nblk;  // the classes, for the second pass (every thread reads what it has written)
    for (int i0 = 0; i0 < a.nblk; i0 += AT * 1024) {
        uint2 r[AT];
#pragma unroll
        for (int u = 0; u < AT; ++u) r[u] = a.span[min(i0 + u * 1024 + t, a.nblk - 1)];
#pragma unroll
        for (int u = 0; u < AT; ++u) {
            const int i = i0 + u * 1024 + t;
            const uint32_t c = i < a.nblk ? class_of(r[u]) : 255u;
            if (i < a.nblk) kind[i] = (uint8_t)c;
            const uint32_t c0 = (uint32_t)uniform((int)c);
            if (__ballot(c == c0) == ~0ull) {  // (neighbours in the index often have the same class)
                if (c0 != 255u && lane == 0) atomicAdd(&hist[c0], 64u);
            } else if (c != 255u) {
                atomicAdd(&hist[c], 1u);
            }
        }
    }
    __syncthreads();
    if (w == 0) {
        // the list: the classes below `split`, all of which the closer bound takes, then that one, of which it takes some
        uint32_t v[4], own = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = hist[4 * lane + i];
            own += v[i];
        }
        uint32_t upto = own;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)upto, dlt);
            if (lane >= dlt) upto += o;
        }
        const uint32_t n = (uint32_t)__shfl((int)upto, 63), near = min((uint32_t)a.near_blocks, n);
        uint32_t before = upto - own;
        if (lane == 0 && near == n) {  // (all of them: no lane finds a class below)
            part[1] = n;
            part[3] = 255u;
            a.near[s] = make_uint4(n, 0u, 0u, 0u);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (near < n && before <= near && before + v[i] > near) {  // (one lane, once: of near < n exactly one class holds that number)
                part[1] = before;
                part[3] = (uint32_t)(4 * lane + i);
                a.near[s] = make_uint4(before, v[i], near - before, 0u);
            }
            before += v[i];
        }
    }
    __syncthreads();
    const uint32_t split = part[3];
    for (int i0 = 0; i0 < a.nblk; i0 += AT * 1024) {
        uint32_t c[AT];
#pragma unroll
        for (int u = 0; u < AT; ++u) c[u] = i0 + u * 1024 + t < a.nblk ? kind[i0 + u * 1024 + t] : 255u;
#pragma unroll
        for (int u = 0; u < AT; ++u) {
            const uint64_t g0 = __ballot(c[u] < split), g1 = __ballot(c[u] == split && c[u] != 255u);
            if ((g0 | g1) == 0ull) continue;
            uint32_t pos = 0u;
            if (lane < 2) pos = atomicAdd(&part[lane], (uint32_t)__popcll(lane == 0 ? g0 : g1));
            const uint64_t mine = c[u] < split ? g0 : g1;
            pos = (uint32_t)__shfl((int)pos, c[u] < split ? 0 : 1);
            if ((mine >> lane) & 1ull)
                list[pos + __builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u))] = (uint16_t)(i0 + u * 1024 + t);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The filter's work: the lists cut into about equal units, a whole number for every sub-tile, as many as give each compute unit one to
// four.  Bound by the latency of one workgroup (313 sub-tiles: 7 us, 625: 11; with a wave for every sub-tile, its count read from memory again and
// 64-bit divisions 16 and 35, which 10 000 queries on a million vectors paid 1 % for).  grid 1, block 1024.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_units(const uint32_t *__restrict__ count, int subs, int block_items, const uint32_t *__restrict__ done,
                                                int subs_per_done, uint32_t *__restrict__ state, uint4 *__restrict__ units,
                                                uint64_t *__restrict__ kept)
{
    __shared__ uint32_t wsum[16], first[1024], many[1024], has[1024];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    auto weight = [&](int i) -> uint32_t { return i < subs && !(done && done[i / subs_per_done] != 0u) ? count[i] : 0u; };
    uint32_t sum = 0u;
    for (int i = t; i < subs; i += 1024) sum += weight(i);
#pragma unroll
    for (int dlt = 32; dlt >= 1; dlt >>= 1) sum += (uint32_t)__shfl_xor((int)sum, dlt);
    if (lane == 0) wsum[w] = sum;
    __syncthreads();
    uint32_t total = 0u;
    for (int i = 0; i < 16; ++i) total += wsum[i];
    // (about 30 000 encodings a unit: staging a sub-tile's tables costs as much as 5000)
    const uint32_t per_cu = min(4u, 1u + (uint32_t)((uint64_t)total * (uint32_t)block_items / (256u * 30000u)));
    const uint32_t most = max(1u, total / (256u * per_cu) + 1u);
    uint32_t base = 0u;
    for (int i0 = 0; i0 < subs; i0 += 1024) {
        const int i = i0 + t;
        const uint32_t n = weight(i), own = (n + most - 1u) / most;
        uint32_t upto = own;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)upto, dlt);
            if (lane >= dlt) upto += o;
        }
        __syncthreads();
        if (lane == 63) wsum[w] = upto;
        __syncthreads();
        uint32_t at = base + upto - own, all = 0u;
        for (int j = 0; j < 16; ++j) {
            at += j < w ? wsum[j] : 0u;
            all += wsum[j];
        }
        first[t] = at;
        many[t] = own;
        has[t] = n;
        // part j of the m parts of the n blocks of sub-tile i (m is at most 1025, as most is more than total / 1024: 32 bits do)
        auto part = [&](uint32_t i, uint32_t n, uint32_t m, uint32_t j) { return make_uint4(i, n * j / m, n * (j + 1u) / m, 0u); };
        // a few units are written by the sub-tile's thread, more by a wave (few sub-tiles of a large index have a hundred each)
        constexpr uint32_t FEW = 8;
        if (own <= FEW)
            for (uint32_t j = 0; j < own; ++j) units[at + j] = part((uint32_t)i, n, own, j);
        __syncthreads();
        for (int k = w; k < 1024 && i0 + k < subs; k += 16) {
            const uint32_t mk = many[k];
            if (mk <= FEW) continue;
            for (uint32_t j = (uint32_t)lane; j < mk; j += 64u) units[first[k] + j] = part((uint32_t)(i0 + k), has[k], mk, j);
        }
        __syncthreads();
        base += all;
    }
    if (t == 0) {
        state[0] = base;
        state[1] = 0u;
        *kept += (uint64_t)total * (uint32_t)block_items;  // (over the batches of a call: etf_last_kept_encodings)
    }
}

}  // namespace etf
