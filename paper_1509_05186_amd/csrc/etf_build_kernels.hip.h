// The index build of up to a few million vectors without a round trip to the host: every kernel finds the counts of
// the ones before it in device memory and computes from them where its arrays lie in the image, so that the host
// launches the whole chain and reads the counts once, at the end.
//
// The sorts are sample sorts.  Every element is (key, tail): the key is the chunks as one integer, first chunk in the
// highest byte, the tail the position (below the id where ids are given), so that no two elements are equal and
// repeated encodings spread over buckets like any others.  One element of each stratum of 128 positions is a sample; a
// sample's rank is counted against all others (k_chain_rank), every eighth in rank is a splitter, an element finds its
// bucket by bisection among the splitters, a workgroup writes its 4096 elements grouped by bucket with the groups'
// bounds (classify), and a workgroup per bucket gathers its groups and sorts them in LDS (bucket_sort): no atomics on
// memory and no slack between buckets.  A bucket expects 1024 elements and LDS holds 4096: more than that needs fewer
// than eight of the 32 samples expected there, about 3e-7 per bucket.  Where it happens all the same (the places of the samples are a fixed function, an input can be made for it)
// the flag `overflow` stops the chain and the host builds by the general path.
//
// Why not a radix sort: eight passes over 8-byte keys (or the twenty launches of a merge sort at these sizes) are bound
// by their launches and their passes over memory; this is four launches and three passes.
//
// A million vectors of 8 chunks in two trees: 1180 us with device-wide library sorts and scans and eleven counts that
// came back to the host between 90 launches, 268 by the chain (10 000: 627 -> 136, five million: 3255 -> 1292; a
// million of 16 chunks in four trees: 2764 -> 578).  The first build after the codebooks were set also lays out their
// copy in pinned memory: 60 to 90 us more.

// ---- keys and elements ------------------------------------------------------------------------------------------

template <int KW> struct KeyOf;
template <> struct KeyOf<1> { using type = uint32_t; };
template <> struct KeyOf<2> { using type = uint64_t; };
template <> struct KeyOf<4> { using type = unsigned __int128; };
template <int KW> using Key = typename KeyOf<KW>::type;

template <int TW> struct TailOf;
template <> struct TailOf<1> { using type = uint32_t; };
template <> struct TailOf<2> { using type = uint64_t; };

// KW key words and TW tail words; in memory KW + TW words, least significant first, tail before key
template <int KW, int TW> struct Elem {
    static constexpr int W = KW + TW;
    Key<KW> key;
    typename TailOf<TW>::type tail;
};

template <int KW, int TW> __device__ __forceinline__ bool less(const Elem<KW, TW> &a, const Elem<KW, TW> &b)
{
    return a.key < b.key || (a.key == b.key && a.tail < b.tail);
}

// words of a value, least significant first
template <typename V> __device__ __forceinline__ uint32_t word_of(V v, int i) { return (uint32_t)(v >> (32 * i)); }

template <int KW> __device__ __forceinline__ Key<KW> key_load(const uint32_t *p)
{
    Key<KW> k = 0;
#pragma unroll
    for (int i = 0; i < KW; ++i) k |= (Key<KW>)p[i] << (32 * i);
    return k;
}

template <int KW> __device__ __forceinline__ void key_store(uint32_t *p, Key<KW> k)
{
#pragma unroll
    for (int i = 0; i < KW; ++i) p[i] = word_of(k, i);
}

template <int KW, int TW> __device__ __forceinline__ Elem<KW, TW> elem_load(const uint32_t *p)
{
    Elem<KW, TW> e;
    e.tail = p[0];
    if constexpr (TW == 2) e.tail |= (uint64_t)p[1] << 32;
    e.key = key_load<KW>(p + TW);
    return e;
}

template <int KW, int TW> __device__ __forceinline__ void elem_store(uint32_t *p, const Elem<KW, TW> &e)
{
#pragma unroll
    for (int i = 0; i < TW; ++i) p[i] = word_of(e.tail, i);
    key_store<KW>(p + TW, e.key);
}

// leading bytes in which two keys agree (4 KW where they are equal)
template <int KW> __device__ __forceinline__ int key_lcp(Key<KW> a, Key<KW> b)
{
    const Key<KW> x = a ^ b;
    if constexpr (KW == 1) return x ? __clz((int)x) >> 3 : 4;
    if constexpr (KW == 2) return x ? __clzll((long long)x) >> 3 : 8;
    if constexpr (KW == 4) {
        const uint64_t hi = (uint64_t)(x >> 64), lo = (uint64_t)x;
        return hi ? __clzll((long long)hi) >> 3 : lo ? 8 + (__clzll((long long)lo) >> 3) : 16;
    }
    return 0;
}

// chunks [c0, c0 + D) of a key as a key of KT words
template <int KW, int KT> __device__ __forceinline__ Key<KT> key_part(Key<KW> k, int c0, int D)
{
    const Key<KT> top = (Key<KT>)((Key<KW>)(k << (8 * c0)) >> (32 * (KW - KT)));
    return top >> (8 * (4 * KT - D)) << (8 * (4 * KT - D));
}

// chunk j of a key
template <int KW> __device__ __forceinline__ uint8_t key_chunk(Key<KW> k, int j) { return (uint8_t)(k >> (8 * (4 * KW - 1 - j))); }

// The first 4 `words` bytes of a key in order (`words` at most the key's).
template <int KW> __device__ __forceinline__ void key_write_front(uint8_t *dst, Key<KW> k, int words)
{
    uint32_t *d = (uint32_t *)dst;
#pragma unroll
    for (int i = 0; i < KW; ++i)
        if (i < words) d[i] = __builtin_bswap32(word_of(k, KW - 1 - i));
}

// Row r of an array of M bytes a row as a key.  Rows of 4 KW bytes are read in words where the array allows (`words`).
template <int KW> __device__ __forceinline__ Key<KW> key_of_row(const uint8_t *rows, int64_t r, int M, bool words)
{
    Key<KW> k = 0;
    if (words) {
        const uint32_t *p = (const uint32_t *)(rows + r * (4 * KW));
#pragma unroll
        for (int i = 0; i < KW; ++i) k |= (Key<KW>)__builtin_bswap32(p[i]) << (32 * (KW - 1 - i));
    } else {
        for (int j = 0; j < M; ++j) k |= (Key<KW>)rows[r * M + j] << (8 * (4 * KW - 1 - j));
    }
    return k;
}

template <int KW> __device__ __forceinline__ void row_of_key(uint8_t *rows, int64_t r, int M, Key<KW> k)
{
    if (M == 4 * KW) {
        key_write_front<KW>(rows + r * (4 * KW), k, KW);
    } else {
        for (int j = 0; j < M; ++j) rows[r * M + j] = key_chunk<KW>(k, j);
    }
}

// ---- arguments --------------------------------------------------------------------------------------------------

constexpr int PREP_NT = 256;   // threads of the kernels that go over rows, samples and draws
constexpr int CLS_NT = 1024;   // ... that deal elements into buckets
constexpr int CLS_TILE = 4096; // elements a workgroup deals
constexpr int RANK_PARTS = 8;  // workgroups that share the comparisons of 64 samples
constexpr int DRAW_TILE = 256;
constexpr int LVL_NT = 1024;   // threads of the level kernels
constexpr int LVL_TILE = 4096; // sub-encodings of a workgroup of the level kernels
constexpr int LVL_CH = LVL_TILE / 64;
constexpr int CATS = 2 * ETF_MAX_M;  // counters of a tile: internal nodes per level, leaves per level

// Counts of a build in device memory; U, nI, nL as the host's, nI and nL by chunk (c0 + level).
struct BuildScal {
    uint32_t Nd, overflow, S_enc, Ainv, max_dup, faults, pad0, pad1;
    uint32_t U[ETF_MAX_M], nI[ETF_MAX_M], nL[ETF_MAX_M];
};

// Arrays of one sort: the elements grouped by bucket within each tile, bounds[tile][bucket] of the groups, the elements
// in order, samples, their ranks; per bucket the elements in it, how many of them differ from their predecessor in the
// bucket (all chunks / tree 0's chunks), and the first and last key.
struct SortBufs {
    uint32_t *grouped, *sorted;
    uint16_t *bounds;
    uint32_t *smp, *rank, *count, *nh, *nh0, *first, *last;
};

struct ChainArgs {
    const uint8_t *codes;
    const int32_t *ids;
    uint32_t N;
    int M, K, T;
    bool permuted, in_words;          // chunk order; the caller's rows can be read in words
    uint8_t src[ETF_MAX_M];
    uint8_t cb[ETF_MAX_M + 1];
    int wshift;                       // log2 of the positions per sample
    uint32_t cap;                     // elements a bucket holds
    uint32_t bstride;                 // bounds of a tile
    int64_t sample_min, sample_scale; // the options behind sample_size
    uint64_t seed;
    // the image: arrays whose places do not depend on counts
    char *img;
    int64_t o_codes, o_ids_in, o_ids_sorted, o_ebegin;
    int64_t n_sample_pos;
    uint64_t A_pos, B_pos;
    int rstride0;
    const uint32_t *tables;           // the quantiser's tables as they stand at the image's start, in host memory
    uint32_t table_words;
    BuildScal *scal_host;             // where the counts go in the end, in host memory
    // workspace
    BuildScal *scal;
    uint32_t *zero;                   // cleared by the first kernel: scal, the samples' ranks
    uint32_t zero_words;
    uint32_t *faults;                 // [workgroups of the first kernel]
    SortBufs s0, st;                  // the vectors; tree 1 (tree t: t - 1 strides further)
    int64_t elem_stride, bounds_stride, smp_stride, rank_stride, bucket_stride, key_stride;
    uint32_t *enc_of_rank;            // [N] distinct encoding of the i-th vector in sorted order
    uint32_t *leaf, *leaf_t;          // [N] leaf of every distinct encoding: tree 0; tree 1 (further ones: as elem_stride)
    uint32_t *dk, *dk_t;              // [N] KT words: the distinct sub-encodings of tree 0; of tree 1 (likewise)
    uint32_t *draw, *kept;            // [S0] encodings drawn for the sample, [tiles] draws kept
    uint32_t *tile_cnt;               // [T][tiles][CATS]
    int lvl_tiles;
};

__device__ __forceinline__ uint32_t *tree_leaf(const ChainArgs &a, int t) { return t == 0 ? a.leaf : a.leaf_t + (t - 1) * a.elem_stride; }
__device__ __forceinline__ uint32_t *tree_dk(const ChainArgs &a, int t) { return t == 0 ? a.dk : a.dk_t + (t - 1) * a.elem_stride; }

__device__ __forceinline__ SortBufs tree_bufs(const ChainArgs &a, int t)
{
    SortBufs s = a.st;
    const int64_t i = t - 1;
    s.grouped += i * a.elem_stride;
    s.sorted += i * a.elem_stride;
    s.bounds += i * a.bounds_stride;
    s.smp += i * a.smp_stride;
    s.rank += i * a.rank_stride;
    s.count += i * a.bucket_stride;
    s.nh += i * a.bucket_stride;
    s.nh0 += i * a.bucket_stride;
    s.first += i * a.key_stride;
    s.last += i * a.key_stride;
    return s;
}

// (a bucket expects a quarter of what it can hold)
__host__ __device__ inline uint32_t n_buckets(uint32_t n, uint32_t cap, int wshift) { return n <= cap / 4 ? 1u : n >> (wshift + 3); }
__host__ __device__ inline uint32_t n_samples(uint32_t n, uint32_t cap, int wshift) { return n <= cap / 4 ? 0u : n >> wshift; }

// position i of n is a sample (its number is i >> wshift)
__device__ __forceinline__ bool is_sample(uint32_t i, uint32_t n, uint32_t cap, int wshift)
{
    const uint32_t s = i >> wshift;
    if (s >= n_samples(n, cap, wshift)) return false;
    const uint32_t m = (1u << wshift) - 1;
    return (i & m) == ((uint32_t)mix64(0x2545F4914F6CDD1Dull ^ s) & m);
}

__host__ __device__ inline int64_t place(int64_t &off, int64_t bytes)
{
    const int64_t o = off;
    off = (off + (bytes > 4 ? bytes : 4) + 255) & ~(int64_t)255;
    return o;
}

// Offsets of the image from `ebegin` on: the same order and rounding as compute_layout (the host compares its own with
// the end that the last kernel would reach by refusing images below the bound).
struct Offsets {
    int64_t enc_of_pos, ecodes, sample_enc, sample_pos, sample_enc_codes, sample_pos_codes, rec0, trees;
};

__device__ inline Offsets offsets(const ChainArgs &a, uint32_t Nd, uint32_t S_enc)
{
    Offsets o;
    int64_t off = a.o_ebegin;
    place(off, ((int64_t)Nd + 1) * 4);
    o.enc_of_pos = place(off, (int64_t)a.N * 4);
    o.ecodes = place(off, (int64_t)Nd * a.M);
    o.sample_enc = place(off, (int64_t)S_enc * 4);
    o.sample_pos = place(off, a.n_sample_pos * 4);
    o.sample_enc_codes = place(off, (int64_t)S_enc * a.M);
    o.sample_pos_codes = place(off, a.n_sample_pos * a.M);
    o.rec0 = place(off, (int64_t)Nd * a.rstride0);
    o.trees = off;
    return o;
}

__device__ inline int tree_depth_class(int D)
{
    int c = 1;
    while (c < D) c <<= 1;
    return c;
}

struct TreeOffsets {
    int64_t rec;
    int64_t icode[ETF_MAX_M], iparent[ETF_MAX_M], lcodes[ETF_MAX_M], lparent[ETF_MAX_M], lrow[ETF_MAX_M];
};

// The arrays of tree t, placed from `off` on: put(array, level, offset), arrays 0 leaf_of, 1 rec, 2 to 6 the levels'.
template <typename F> __device__ inline void place_tree(const ChainArgs &a, const BuildScal &scal, int t, int64_t &off, F put)
{
    const int c0 = a.cb[t], D = a.cb[t + 1] - c0, c = tree_depth_class(D);
    if (a.T > 1) put(0, 0, place(off, (int64_t)scal.Nd * 4));
    put(1, 0, place(off, (int64_t)scal.U[t] * (c < 4 ? 4 : c)));
    for (int l = 0; l < D; ++l) {
        const int64_t nI = scal.nI[c0 + l], nL = scal.nL[c0 + l];
        put(2, l, place(off, nI));
        put(3, l, place(off, nI * 4));
        put(4, l, place(off, nL * ((D - l + 3) & ~3)));
        put(5, l, place(off, nL * 4));
        put(6, l, place(off, nL * 4));
    }
}

// the counts in LDS, read by a whole workgroup (a loop over them in memory would wait for one load after the other)
__device__ inline void load_counts(const BuildScal *from, BuildScal &to)
{
    constexpr int n = sizeof(BuildScal) / 4;
    if (threadIdx.x < n) ((uint32_t *)&to)[threadIdx.x] = ((const uint32_t *)from)[threadIdx.x];
    __syncthreads();
}

// ---- the first kernel: input into the image, its faults, the samples of the vectors ------------------------------
// Bound by memory: 8 M bytes and ids in and out once.
template <int KW, int TW>
__global__ void __launch_bounds__(PREP_NT) k_chain_prep(ChainArgs a)
{
    const uint32_t i = blockIdx.x * PREP_NT + threadIdx.x;
    for (uint32_t j = i; j < a.zero_words; j += gridDim.x * PREP_NT) a.zero[j] = 0;
    uint8_t *rows = (uint8_t *)(a.img + a.o_codes);
    int bad = 0;
    if (i < a.N) {
        Key<KW> k;
        if (a.permuted) {
            k = 0;
            for (int j = 0; j < a.M; ++j) k |= (Key<KW>)a.codes[(int64_t)i * a.M + a.src[j]] << (8 * (4 * KW - 1 - j));
        } else {
            k = key_of_row<KW>(a.codes, i, a.M, a.in_words);
        }
        const int32_t id = a.ids ? a.ids[i] : (int32_t)i;
        if (rows != a.codes || a.permuted) row_of_key<KW>(rows, i, a.M, k);
        ((int32_t *)(a.img + a.o_ids_in))[i] = id;
        if (a.K < 256)
            for (int j = 0; j < a.M; ++j)
                if (key_chunk<KW>(k, j) >= a.K) bad = 1;
        if (id < 0) bad |= 2;
        if (is_sample(i, a.N, a.cap, a.wshift)) {
            Elem<KW, TW> e;
            e.key = k;
            e.tail = i;
            if constexpr (TW == 2) e.tail |= (uint64_t)(uint32_t)id << 32;
            elem_store<KW, TW>(a.s0.smp + (int64_t)(i >> a.wshift) * (KW + TW), e);
        }
    }
    const int b1 = __syncthreads_or(bad & 1), b2 = __syncthreads_or(bad & 2);
    if (threadIdx.x == 0) a.faults[blockIdx.x] = (b1 ? 1u : 0u) | (b2 ? 2u : 0u);
}

// ---- ranks of the samples ----------------------------------------------------------------------------------------
// Workgroup (g, p) compares samples 64 g .. 64 g + 63, one per lane, with the p-th part of all samples, which a wave
// reads with scalar loads.  Without ids, positions ascend with the sample's number, so that of two equal keys the lower
// number comes first: samples before the 64 count where their key is not larger, those behind where it is smaller.
// Bound by vector issue: S^2 comparisons of two to three instructions.
template <int KW, int TW>
__device__ void rank_samples(const uint32_t *__restrict__ smp, uint32_t *rank, uint32_t S, uint32_t blk)
{
    constexpr int W = KW + TW;
    __shared__ uint32_t part[PREP_NT / 64][64];
    const uint32_t g = blk / RANK_PARTS;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t slice = (blk % RANK_PARTS) * (PREP_NT / 64) + wave;
    constexpr uint32_t SLICES = RANK_PARTS * (PREP_NT / 64);
    const uint32_t i = g * 64 + lane;
    uint32_t lo = (uint32_t)((uint64_t)S * slice / SLICES), hi = (uint32_t)((uint64_t)S * (slice + 1) / SLICES);
    lo = __builtin_amdgcn_readfirstlane((int)lo);
    hi = __builtin_amdgcn_readfirstlane((int)hi);
    const Elem<KW, TW> me = elem_load<KW, TW>(smp + (int64_t)min(i, S - 1) * W);
    uint32_t r = 0;
    if constexpr (TW == 1) {
        const uint32_t m0 = min(max(g * 64, lo), hi), m1 = min(max(g * 64 + 64, lo), hi);
#pragma unroll 8
        for (uint32_t j = lo; j < m0; ++j) r += key_load<KW>(smp + (int64_t)j * W + TW) <= me.key ? 1u : 0u;
        for (uint32_t j = m0; j < m1; ++j) {
            const Key<KW> k = key_load<KW>(smp + (int64_t)j * W + TW);
            r += (k < me.key || (k == me.key && j < i)) ? 1u : 0u;
        }
#pragma unroll 8
        for (uint32_t j = m1; j < hi; ++j) r += key_load<KW>(smp + (int64_t)j * W + TW) < me.key ? 1u : 0u;
    } else {
#pragma unroll 4
        for (uint32_t j = lo; j < hi; ++j) r += less(elem_load<KW, TW>(smp + (int64_t)j * W), me) ? 1u : 0u;
    }
    part[wave][lane] = r;
    __syncthreads();
    if (wave == 0 && i < S) {
        for (int w = 1; w < PREP_NT / 64; ++w) r += part[w][lane];
        if (r) atomicAdd(&rank[i], r);
    }
}

template <int KW, int TW>
__global__ void __launch_bounds__(PREP_NT) k_chain_rank(ChainArgs a)
{
    rank_samples<KW, TW>(a.s0.smp, a.s0.rank, n_samples(a.N, a.cap, a.wshift), blockIdx.x);
}

// ---- elements into buckets ---------------------------------------------------------------------------------------
// LDS: the splitters as W arrays of `stride` words, then a count per bucket.  Bound by latency: the bisection's ten to
// twelve dependent reads, four elements per thread in flight.  (Slabs that the workgroups filled through an atomic per
// bucket and workgroup: 40 us for a million elements, most of it the atomics.)
// elem(i): the i-th of n elements.
template <int KW, int TW, typename F>
__device__ void classify(const SortBufs &s, uint32_t n, uint32_t cap, int wshift, uint32_t stride, uint32_t bstride, uint32_t *lds, F elem)
{
    constexpr int W = KW + TW, PER = CLS_TILE / CLS_NT;
    __shared__ uint32_t wave_sum[CLS_NT / 64];
    const uint32_t B = n_buckets(n, cap, wshift), S = n_samples(n, cap, wshift);
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint32_t *cnt = lds + W * stride;
    Elem<KW, TW> e[PER];
    uint32_t b[PER], slot[PER];
    const uint32_t i0 = blockIdx.x * CLS_TILE + t;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        e[q] = elem(min(i0 + q * CLS_NT, n - 1));
        b[q] = 0;
    }
    for (uint32_t x = t; x < B; x += CLS_NT) cnt[x] = 0;
    for (uint32_t i = t; i < S; i += 4 * CLS_NT) {   // (four samples requested at once, wanted or not)
        uint32_t r[4], w[4][W];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t j = min(i + q * CLS_NT, S - 1);
            r[q] = s.rank[j];
#pragma unroll
            for (int x = 0; x < W; ++x) w[q][x] = s.smp[(int64_t)j * W + x];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if ((r[q] & 7u) == 0 && r[q] > 0 && (r[q] >> 3) < B)
#pragma unroll
                for (int x = 0; x < W; ++x) lds[x * stride + (r[q] >> 3) - 1] = w[q][x];
    }
    __syncthreads();
    uint32_t step = 1;
    while (step * 2 <= B - 1) step *= 2;
    if (B > 1)
        for (; step > 0; step >>= 1)
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const uint32_t at = b[q] + step - 1;   // the splitter that closes the next `step` buckets
                if (at >= B - 1) continue;
                uint32_t w[W];
#pragma unroll
                for (int x = 0; x < W; ++x) w[x] = lds[x * stride + at];
                if (!less(e[q], elem_load<KW, TW>(w))) b[q] += step;
            }
#pragma unroll
    for (int q = 0; q < PER; ++q) slot[q] = i0 + q * CLS_NT < n ? atomicAdd(&cnt[b[q]], 1u) : 0u;
    __syncthreads();
    // counts to bounds: a thread sums `per` buckets, then waves and workgroup
    const uint32_t per = (B + CLS_NT - 1) / CLS_NT, b0 = min(t * per, B), b1 = min(b0 + per, B);
    uint32_t own = 0;
    for (uint32_t x = b0; x < b1; ++x) own += cnt[x];
    uint32_t incl = own;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o);
        if ((int)lane >= o) incl += y;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t at = incl - own;
    for (uint32_t w = 0; w < wave; ++w) at += wave_sum[w];
    uint16_t *bounds = s.bounds + (int64_t)blockIdx.x * bstride;
    for (uint32_t x = b0; x < b1; ++x) {
        const uint32_t c = cnt[x];
        cnt[x] = at;
        bounds[x] = (uint16_t)at;
        at += c;
    }
    if (t == CLS_NT - 1) bounds[B] = (uint16_t)at;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (i0 + q * CLS_NT < n)
            elem_store<KW, TW>(s.grouped + ((int64_t)blockIdx.x * CLS_TILE + cnt[b[q]] + slot[q]) * W, e[q]);
}

template <int KW, int TW>
__global__ void __launch_bounds__(CLS_NT) k_chain_classify(ChainArgs a, uint32_t stride)
{
    extern __shared__ uint32_t blds[];
    const uint8_t *rows = (const uint8_t *)(a.img + a.o_codes);
    const int32_t *ids = (const int32_t *)(a.img + a.o_ids_in);
    classify<KW, TW>(a.s0, a.N, a.cap, a.wshift, stride, a.bstride, blds, [&](uint32_t i) {
        Elem<KW, TW> e;
        e.key = key_of_row<KW>(rows, i, a.M, a.M == 4 * KW);
        e.tail = i;
        if constexpr (TW == 2) e.tail |= (uint64_t)(uint32_t)ids[i] << 32;
        return e;
    });
}

// ---- a bucket sorted in LDS --------------------------------------------------------------------------------------
// The workgroup gathers its group of every tile and sorts by sampling once more: every eighth element is a splitter,
// elements are dealt into the parts between them, about eight to a part, and an element's rank in its part is counted
// against all others there.  58 us for a million elements of 12 bytes, the gather included, bound by latency (two dependent reads of memory,
// some thirty of LDS, ten barriers: 50 000 clocks for a workgroup with two others on its CU) and comparisons: a third of
// the issue slots.  (Merging sorted runs pairwise, eight rounds of twenty dependent reads each, took 51 us for a million
// elements that lay side by side, in slabs whose filling took 40 us more than the tiles' groups do; with LDS for 2048
// elements and the larger buckets in two halves 91, the halves of a single bucket one after the other.)
// Words lie in W separate arrays.
template <int KW, int TW> __device__ __forceinline__ Elem<KW, TW> lds_elem(const uint32_t *lds, uint32_t stride, uint32_t i)
{
    constexpr int W = KW + TW;
    uint32_t w[W];
#pragma unroll
    for (int x = 0; x < W; ++x) w[x] = lds[x * stride + i];
    return elem_load<KW, TW>(w);
}

template <int KW, int TW> __device__ __forceinline__ void lds_put(uint32_t *lds, uint32_t stride, uint32_t i, const Elem<KW, TW> &e)
{
    constexpr int W = KW + TW;
    uint32_t w[W];
    elem_store<KW, TW>(w, e);
#pragma unroll
    for (int x = 0; x < W; ++x) lds[x * stride + i] = w[x];
}

// Workgroups go to the eight XCDs in turn: an XCD takes a stretch of the buckets, since neighbouring buckets' groups share
// the lines of a tile (65 against 61 us for a million elements).
__device__ __forceinline__ uint32_t bucket_of_block(uint32_t block, uint32_t B) { return (block & 7u) * ((B + 7) / 8) + (block >> 3); }

constexpr int MAX_SPLIT = 192;  // (with 256 the LDS of three workgroups of 4096 elements of three words is a little more than a CU has)

template <int KW, int TW, int NT, uint32_t CAP>
__device__ void bucket_sort(const SortBufs &s, uint32_t n, uint32_t bstride, uint32_t bucket, int D0, BuildScal *scal, uint32_t *lds)
{
    constexpr int W = KW + TW, PER = CAP / NT;
    __shared__ uint32_t heads[2], off_sum, wave_sum[NT / 64], rank[MAX_SPLIT], part_begin[MAX_SPLIT + 2];
    __shared__ uint32_t split[W * MAX_SPLIT];
    using E = Elem<KW, TW>;
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6, tiles = (n + CLS_TILE - 1) / CLS_TILE;
    if (t < 2) heads[t] = 0;
    if (t == 2) off_sum = 0;
    for (uint32_t i = t; i < MAX_SPLIT + 2; i += NT) {
        part_begin[i] = 0;
        if (i < MAX_SPLIT) rank[i] = 0;
    }
    __syncthreads();
    // Where every tile's group starts in the bucket (the elements' LDS is still free); what the tiles hold before the
    // bucket, summed, is its place in the whole order.
    uint32_t *group_at = lds;
    uint16_t *group_from = (uint16_t *)(lds + tiles);
    uint32_t cnt = 0, before = 0;
    for (uint32_t t0 = 0; t0 < tiles; t0 += NT) {
        const uint32_t tile = t0 + t;
        uint32_t lo = 0, hi = 0;
        if (tile < tiles) {
            lo = s.bounds[(int64_t)tile * bstride + bucket];
            hi = s.bounds[(int64_t)tile * bstride + bucket + 1];
        }
        before += lo;
        uint32_t incl = hi - lo;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o);
            if ((int)lane >= o) incl += y;
        }
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        uint32_t at = cnt + incl - (hi - lo);
        for (uint32_t w = 0; w < NT / 64; ++w) {
            if (w < wave) at += wave_sum[w];
            cnt += wave_sum[w];
        }
        __syncthreads();
        if (tile < tiles) {
            group_at[tile] = at;
            group_from[tile] = (uint16_t)lo;
        }
    }
    for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
    if (lane == 0 && before) atomicAdd(&off_sum, before);
    if (t == 0) s.count[bucket] = cnt;
    __syncthreads();
    if (cnt > CAP) {
        if (t == 0) scal->overflow = 1;
        return;
    }
    if (cnt == 0) {
        if (t == 0) s.nh[bucket] = s.nh0[bucket] = 0;
        return;
    }
    // an element's tile by bisection: the last one that starts at or before it
    E e[PER];
    {
        uint32_t tl[PER], step = 1;
        while (step * 2 <= tiles - 1) step *= 2;
#pragma unroll
        for (int q = 0; q < PER; ++q) tl[q] = 0;
        for (; step > 0; step >>= 1)
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if (q * NT < cnt) {
                    const uint32_t at = tl[q] + step;
                    if (at < tiles && group_at[at] <= min(q * NT + t, cnt - 1)) tl[q] = at;
                }
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (q * NT < cnt) {
                const uint32_t at = tl[q] * CLS_TILE + group_from[tl[q]] + min(q * NT + t, cnt - 1) - group_at[tl[q]];
                e[q] = elem_load<KW, TW>(s.grouped + (int64_t)at * W);
            }
    }
    __syncthreads();
    // splitters: elements 0, stride, 2 stride, ... in order of their rank
    const uint32_t ns = min(max(cnt / 8, 1u), (uint32_t)MAX_SPLIT), stride = cnt / ns, groups = (ns + 63) / 64, slices = NT / 64 / groups;
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (q * NT + t < cnt) {
            const uint32_t j = (q * NT + t) / stride;
            if (j < ns && j * stride == q * NT + t) lds_put(lds, MAX_SPLIT, j, e[q]);
        }
    __syncthreads();
    {
        const uint32_t i = (wave % groups) * 64 + lane, slice = wave / groups;
        if (slice < slices) {
            const E me = lds_elem<KW, TW>(lds, MAX_SPLIT, min(i, ns - 1));
            uint32_t r = 0;
#pragma unroll 8
            for (uint32_t j = ns * slice / slices; j < ns * (slice + 1) / slices; ++j)
                r += less(lds_elem<KW, TW>(lds, MAX_SPLIT, j), me) ? 1u : 0u;
            if (i < ns && r) atomicAdd(&rank[i], r);
        }
    }
    __syncthreads();
    if (t < ns) lds_put(split, MAX_SPLIT, rank[t], lds_elem<KW, TW>(lds, MAX_SPLIT, t));
    __syncthreads();
    uint32_t part[PER], slot[PER], step = 1;
    while (step * 2 <= ns) step *= 2;
#pragma unroll
    for (int q = 0; q < PER; ++q) part[q] = 0;
    for (; step > 0; step >>= 1)
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (q * NT < cnt) {
                const uint32_t at = part[q] + step - 1;
                if (at < ns && !less(e[q], lds_elem<KW, TW>(split, MAX_SPLIT, at))) part[q] += step;
            }
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (q * NT + t < cnt) slot[q] = atomicAdd(&part_begin[part[q] + 1], 1u);
    __syncthreads();
    if (t < 64) {   // counts of parts 0 .. ns stand at 1 .. ns + 1; 0 stays 0
        uint32_t sum = 0;
        for (uint32_t c = 0; c <= ns; c += 64) {
            const uint32_t x = c + lane <= ns ? part_begin[c + lane + 1] : 0;
            uint32_t incl = x;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(incl, o);
                if ((int)lane >= o) incl += y;
            }
            if (c + lane <= ns) part_begin[c + lane + 1] = sum + incl;
            sum += __shfl(incl, 63);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (q * NT + t < cnt) lds_put(lds, CAP, part_begin[part[q]] + slot[q], e[q]);
    __syncthreads();
    // ranks in the order of the parts: the lanes of a wave then read a few parts, the same element for many lanes (58
    // against 61 us with the elements in the order they came)
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (q * NT + t < cnt) {
            const uint32_t i = q * NT + t;
            uint32_t p = 0;   // the last part that starts at or before i
            for (uint32_t step = 128; step > 0; step >>= 1)
                if (p + step <= ns && part_begin[p + step] <= i) p += step;
            e[q] = lds_elem<KW, TW>(lds, CAP, i);
            const uint32_t p0 = part_begin[p], p1 = part_begin[p + 1];
            uint32_t r = p0;
#pragma unroll 4
            for (uint32_t j = p0; j < p1; ++j) r += less(lds_elem<KW, TW>(lds, CAP, j), e[q]) ? 1u : 0u;
            slot[q] = r;
        }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (q * NT + t < cnt) lds_put(lds, CAP, slot[q], e[q]);
    __syncthreads();
    uint32_t *out = s.sorted + (int64_t)off_sum * W;
    uint32_t h = 0, h0 = 0;
    for (uint32_t i = t; i < cnt; i += NT) {
        const E x = lds_elem<KW, TW>(lds, CAP, i);
        elem_store<KW, TW>(out + (int64_t)i * W, x);
        if (i == 0) key_store<KW>(s.first + (int64_t)bucket * KW, x.key);
        if (i == cnt - 1) key_store<KW>(s.last + (int64_t)bucket * KW, x.key);
        if (i > 0) {
            const int p = key_lcp<KW>(x.key, lds_elem<KW, TW>(lds, CAP, i - 1).key);
            h += p < 4 * KW ? 1u : 0u;
            h0 += p < D0 ? 1u : 0u;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        h += __shfl_xor(h, o);
        h0 += __shfl_xor(h0, o);
    }
    if (lane == 0) {
        atomicAdd(&heads[0], h);
        atomicAdd(&heads[1], h0);
    }
    __syncthreads();
    if (t == 0) {
        s.nh[bucket] = heads[0];
        s.nh0[bucket] = heads[1];
    }
}

template <int KW, int TW, int NT, uint32_t CAP>
__global__ void __launch_bounds__(NT) k_chain_sort(ChainArgs a)
{
    extern __shared__ uint32_t blds[];
    const uint32_t B = n_buckets(a.N, a.cap, a.wshift), bucket = bucket_of_block(blockIdx.x, B);
    if ((blockIdx.x >> 3) >= (B + 7) / 8 || bucket >= B) return;
    bucket_sort<KW, TW, NT, CAP>(a.s0, a.N, a.bstride, bucket, a.cb[1], a.scal, blds);
}

// ---- where a bucket's elements and its distinct keys stand in the whole order ------------------------------------
struct BucketPlace {
    uint32_t off, hd, hd0;    // elements, distinct keys, distinct prefixes of D0 chunks in the buckets before
    uint32_t tot, tot0;       // distinct keys and prefixes in all buckets
    uint32_t edge, edge0;     // the bucket's first element differs from the one before it
};

template <int KW, int NT>
__device__ BucketPlace bucket_place(const SortBufs &s, uint32_t B, uint32_t bucket, int D0)
{
    __shared__ uint32_t acc[7];
    if (threadIdx.x < 7) acc[threadIdx.x] = 0;
    __syncthreads();
    uint32_t v[5] = {0, 0, 0, 0, 0};
    for (uint32_t b = threadIdx.x; b < B; b += NT) {
        // (everything requested at once; an empty bucket before this one is rare)
        const uint32_t c = s.count[b], nh = s.nh[b], nh0 = s.nh0[b], cp = s.count[b > 0 ? b - 1 : 0];
        const Key<KW> first = key_load<KW>(s.first + (int64_t)b * KW);
        Key<KW> last = key_load<KW>(s.last + (int64_t)(b > 0 ? b - 1 : 0) * KW);
        if (c == 0) continue;
        int64_t p = (int64_t)b - 1;
        if (p >= 0 && cp == 0) {
            while (p >= 0 && s.count[p] == 0) --p;
            if (p >= 0) last = key_load<KW>(s.last + p * KW);
        }
        uint32_t edge = 1, edge0 = 1;
        if (p >= 0) {
            const int n = key_lcp<KW>(first, last);
            edge = n < 4 * KW ? 1u : 0u;
            edge0 = n < D0 ? 1u : 0u;
        }
        const uint32_t h = nh + edge, h0 = nh0 + edge0;
        if (b < bucket) {
            v[0] += c;
            v[1] += h;
            v[2] += h0;
        }
        v[3] += h;
        v[4] += h0;
        if (b == bucket) {
            acc[5] = edge;
            acc[6] = edge0;
        }
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        for (int o = 32; o > 0; o >>= 1) v[i] += __shfl_xor(v[i], o);
        if ((threadIdx.x & 63) == 0 && v[i]) atomicAdd(&acc[i], v[i]);
    }
    __syncthreads();
    BucketPlace r;
    r.off = acc[0]; r.hd = acc[1]; r.hd0 = acc[2]; r.tot = acc[3]; r.tot0 = acc[4]; r.edge = acc[5]; r.edge0 = acc[6];
    return r;
}

// The bucket's elements in order, 64 per wave step, with the number of distinct keys (and prefixes) up to and
// including each: emit(i, element, head, rank, head0, rank0), ranks counted from the whole order's start.
template <int KW, int TW, int NT, typename F>
__device__ void bucket_walk(const SortBufs &s, uint32_t bucket, int D0, const BucketPlace &pl, F emit)
{
    constexpr int W = KW + TW, CH = NT / 8;  // chunks of 64 elements in a full bucket
    __shared__ uint64_t mask[CH], mask0[CH];
    __shared__ uint32_t pre[CH], pre0[CH];
    constexpr uint32_t CAP = NT * 8;
    const uint32_t cnt = min(s.count[bucket], CAP), lane = threadIdx.x & 63;
    const uint32_t *run = s.sorted + (int64_t)pl.off * W;
    const uint32_t nch = (cnt + 63) / 64;
    for (uint32_t c = threadIdx.x >> 6; c < nch; c += NT / 64) {
        const uint32_t i = c * 64 + lane;
        bool h = false, h0 = false;
        if (i < cnt) {
            if (i == 0) {
                h = pl.edge != 0;
                h0 = pl.edge0 != 0;
            } else {
                const int n = key_lcp<KW>(key_load<KW>(run + (int64_t)i * W + TW), key_load<KW>(run + (int64_t)(i - 1) * W + TW));
                h = n < 4 * KW;
                h0 = n < D0;
            }
        }
        const uint64_t m = __ballot(h), m0 = __ballot(h0);
        if (lane == 0) {
            mask[c] = m;
            mask0[c] = m0;
        }
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        uint32_t h = pl.hd, h0 = pl.hd0;
        for (uint32_t c0 = 0; c0 < nch; c0 += 64) {
            const uint32_t c = c0 + lane;
            const uint32_t n = c < nch ? (uint32_t)__popcll(mask[c]) : 0, n0 = c < nch ? (uint32_t)__popcll(mask0[c]) : 0;
            uint32_t x = n, x0 = n0;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(x, o), y0 = __shfl_up(x0, o);
                if ((int)lane >= o) {
                    x += y;
                    x0 += y0;
                }
            }
            if (c < nch) {
                pre[c] = h + x - n;
                pre0[c] = h0 + x0 - n0;
            }
            h += __shfl(x, 63);
            h0 += __shfl(x0, 63);
        }
    }
    __syncthreads();
    for (uint32_t c = threadIdx.x >> 6; c < nch; c += NT / 64) {
        const uint32_t i = c * 64 + lane;
        if (i >= cnt) continue;
        const uint64_t upto = ~0ull >> (63 - lane), m = mask[c], m0 = mask0[c];
        emit(i, elem_load<KW, TW>(run + (int64_t)i * W), (m >> lane & 1) != 0, pre[c] + (uint32_t)__popcll(m & upto), (m0 >> lane & 1) != 0,
             pre0[c] + (uint32_t)__popcll(m0 & upto));
    }
}

// ---- the encodings: ids, ranges, numbers, tree 0's leaves, the samples of the other trees ------------------------
// Bound by memory: the scattered 4-byte stores of enc_of_pos are a line each.
template <int KW, int TW, int KT, int NT>
__global__ void __launch_bounds__(NT) k_chain_encodings(ChainArgs a)
{
    if (a.scal->overflow) return;
    const uint32_t B = n_buckets(a.N, a.cap, a.wshift);
    const int D0 = a.cb[1];
    const BucketPlace pl = bucket_place<KW, NT>(a.s0, B, blockIdx.x, D0);
    const uint32_t Nd = pl.tot;
    const Offsets o = offsets(a, Nd, 0);   // (only what lies before the samples is used)
    int32_t *ids_sorted = (int32_t *)(a.img + a.o_ids_sorted);
    uint32_t *ebegin = (uint32_t *)(a.img + a.o_ebegin), *enc_of_pos = (uint32_t *)(a.img + o.enc_of_pos);
    uint8_t *ecodes = (uint8_t *)(a.img + o.ecodes);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.scal->Nd = Nd;
        a.scal->U[0] = pl.tot0;
        ebegin[Nd] = a.N;
    }
    bucket_walk<KW, TW, NT>(a.s0, blockIdx.x, D0, pl, [&](uint32_t i, const Elem<KW, TW> &x, bool head, uint32_t rank, bool head0, uint32_t rank0) {
        const uint32_t e = rank - 1, pos = (uint32_t)x.tail, at = pl.off + i;
        ids_sorted[at] = TW == 2 ? (int32_t)((uint64_t)x.tail >> 32) : (int32_t)pos;
        enc_of_pos[pos] = e;
        a.enc_of_rank[at] = e;
        if (!head) return;
        ebegin[e] = at;
        row_of_key<KW>(ecodes, e, a.M, x.key);
        a.leaf[e] = rank0 - 1;
        if (head0) key_store<KT>(a.dk + (int64_t)(rank0 - 1) * KT, key_part<KW, KT>(x.key, 0, D0));
        if (a.T > 1 && is_sample(e, Nd, a.cap, a.wshift))
            for (int t = 1; t < a.T; ++t) {
                Elem<KT, 1> y;
                y.key = key_part<KW, KT>(x.key, a.cb[t], a.cb[t + 1] - a.cb[t]);
                y.tail = e;
                elem_store<KT, 1>(tree_bufs(a, t).smp + (int64_t)(e >> a.wshift) * (KT + 1), y);
            }
    });
}

// ---- nodes per level ---------------------------------------------------------------------------------------------
constexpr int LVL_PER = LVL_CH / (LVL_NT / 64);  // chunks of 64 sub-encodings of a wave: wave w has w, w + 16, ...

// The wave's sub-encodings of a tile of tree t (0 beyond the last) and how far their neighbours agree with them.
template <int KT> struct Subs {
    Key<KT> k[LVL_PER];
    int x[LVL_PER], y[LVL_PER];
};

template <int KT> __device__ __forceinline__ Subs<KT> load_subs(const uint32_t *dk, uint32_t tile, uint32_t U, int D)
{
    Subs<KT> s;
    Key<KT> before[LVL_PER], after[LVL_PER];
#pragma unroll
    for (int q = 0; q < LVL_PER; ++q) {
        const uint32_t u = min(tile * LVL_TILE + (q * (LVL_NT / 64) + (threadIdx.x >> 6)) * 64 + (threadIdx.x & 63), U - 1);
        s.k[q] = key_load<KT>(dk + (int64_t)u * KT);
        before[q] = key_load<KT>(dk + (int64_t)(u > 0 ? u - 1 : 0) * KT);
        after[q] = key_load<KT>(dk + (int64_t)min(u + 1, U - 1) * KT);
    }
#pragma unroll
    for (int q = 0; q < LVL_PER; ++q) {
        const uint32_t u = tile * LVL_TILE + (q * (LVL_NT / 64) + (threadIdx.x >> 6)) * 64 + (threadIdx.x & 63);
        s.x[q] = u > 0 ? min(D, key_lcp<KT>(s.k[q], before[q])) : 0;
        s.y[q] = u + 1 < U ? min(D, key_lcp<KT>(s.k[q], after[q])) : 0;
    }
    return s;
}

// A prefix group of length l starts at u where a < l; it is an internal node where the next sub-encoding still shares
// it (b >= l, below the last level); u is a leaf of the level at which it is alone in its group, 1 + max(a, b).
__device__ __forceinline__ bool is_internal(int a, int b, int l, int D) { return l < D && a < l && b >= l; }
__device__ __forceinline__ bool is_leaf(int a, int b, int l) { return 1 + max(a, b) == l; }

template <int KT> __device__ void count_levels(const ChainArgs &a, int t, uint32_t tile)
{
    __shared__ uint32_t acc[CATS];
    const uint32_t U = a.scal->U[t], lane = threadIdx.x & 63;
    if (tile * (uint32_t)LVL_TILE >= U) return;
    const int c0 = a.cb[t], D = a.cb[t + 1] - c0;
    const uint32_t *dk = tree_dk(a, t);
    if (threadIdx.x < CATS) acc[threadIdx.x] = 0;
    __syncthreads();
    const Subs<KT> s = load_subs<KT>(dk, tile, U, D);
    uint32_t mine = 0;  // lane c: category c
#pragma unroll
    for (int q = 0; q < LVL_PER; ++q) {
        const bool on = tile * LVL_TILE + (q * (LVL_NT / 64) + (threadIdx.x >> 6)) * 64 + lane < U;
        for (int l = 1; l <= D; ++l) {
            const uint32_t ni = (uint32_t)__popcll(__ballot(on && is_internal(s.x[q], s.y[q], l, D))), nl = (uint32_t)__popcll(__ballot(on && is_leaf(s.x[q], s.y[q], l)));
            mine += (int)lane == l - 1 ? ni : (int)lane == ETF_MAX_M + l - 1 ? nl : 0;
        }
    }
    if (lane < CATS && mine) atomicAdd(&acc[lane], mine);
    __syncthreads();
    if (threadIdx.x < CATS) {
        const uint32_t n = acc[threadIdx.x];
        a.tile_cnt[((int64_t)t * a.lvl_tiles + tile) * CATS + threadIdx.x] = n;
        const int l = threadIdx.x % ETF_MAX_M;
        if (n) atomicAdd(threadIdx.x < ETF_MAX_M ? &a.scal->nI[c0 + l] : &a.scal->nL[c0 + l], n);
    }
}

// ---- draws of the threshold sample, the longest id range, the input's faults -------------------------------------
// sample_size of the host; n_sample_pos is that of N >= Nd vectors, and what the arrays of draws have room for
__device__ inline uint32_t sample_draws(const ChainArgs &a, uint32_t Nd)
{
    const int64_t n = (int64_t)((double)a.sample_scale * sqrt((double)Nd));
    const int64_t s = n > a.sample_min ? n : a.sample_min;
    return (uint32_t)min(min(s, a.n_sample_pos), (int64_t)Nd);
}

// the encoding of the vector drawn from stratum s of S0
__device__ inline uint32_t chain_draw(const ChainArgs &a, uint64_t S0, uint64_t s)
{
    const uint64_t N = a.N, lo = s * N / S0, hi = (s + 1) * N / S0;
    return a.enc_of_rank[lo + mix64(a.seed ^ s) % (hi - lo)];
}

__device__ void draw_sample(const ChainArgs &a, uint32_t blk, uint32_t nblk)
{
    __shared__ uint32_t d[DRAW_TILE + 1], most, kept;
    const uint32_t Nd = a.scal->Nd, S0 = sample_draws(a, Nd);
    // the longest range of ids, a slice of the encodings per workgroup
    if (threadIdx.x == 0) most = kept = 0;
    __syncthreads();
    const uint32_t *ebegin = (const uint32_t *)(a.img + a.o_ebegin);
    uint32_t n = 0, bad = 0;
    for (uint32_t e = blk * PREP_NT + threadIdx.x; e < Nd; e += nblk * PREP_NT) n = max(n, ebegin[e + 1] - ebegin[e]);
    for (uint32_t i = blk * PREP_NT + threadIdx.x; i < (a.N + PREP_NT - 1) / PREP_NT; i += nblk * PREP_NT) bad |= a.faults[i];
    for (int o = 32; o > 0; o >>= 1) n = max(n, (uint32_t)__shfl_xor((int)n, o));
    if ((threadIdx.x & 63) == 0) atomicMax(&most, n);
    if (bad) atomicOr(&a.scal->faults, bad);
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(&a.scal->max_dup, most);
    for (uint32_t tile = blk; tile * (uint32_t)DRAW_TILE < S0; tile += nblk) {
        const uint32_t s0 = tile * DRAW_TILE;
        __syncthreads();
        for (uint32_t i = threadIdx.x; i <= DRAW_TILE; i += PREP_NT) {   // d[i] = draw s0 + i - 1
            const uint32_t s = s0 + i - 1;
            if (s0 + i == 0 || s >= S0) continue;
            d[i] = chain_draw(a, S0, s);
            if (i > 0) a.draw[s] = d[i];
        }
        if (threadIdx.x == 0) kept = 0;
        __syncthreads();
        uint32_t c = 0;
        for (uint32_t i = threadIdx.x; i < DRAW_TILE; i += PREP_NT) {
            const uint32_t s = s0 + i;
            c += s < S0 && (s == 0 || d[i + 1] != d[i]) ? 1u : 0u;
        }
        for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
        if ((threadIdx.x & 63) == 0) atomicAdd(&kept, c);
        __syncthreads();
        if (threadIdx.x == 0) a.kept[tile] = kept;
    }
}

// blockIdx.y < T - 1: ranks of the samples of tree y + 1; T - 1: draws; T: the tables
template <int KT>
__global__ void __launch_bounds__(PREP_NT) k_chain_mid(ChainArgs a, uint32_t draw_blocks)
{
    if (a.scal->overflow) return;
    const int y = (int)blockIdx.y;
    if (y < a.T - 1) {
        const uint32_t S = n_samples(a.scal->Nd, a.cap, a.wshift);
        if (blockIdx.x / RANK_PARTS * 64 >= S) return;
        const SortBufs s = tree_bufs(a, y + 1);
        rank_samples<KT, 1>(s.smp, s.rank, S, blockIdx.x);
    } else if (y == a.T - 1) {
        if (blockIdx.x < draw_blocks) draw_sample(a, blockIdx.x, draw_blocks);
    } else {
        for (uint32_t j = blockIdx.x * PREP_NT + threadIdx.x; j < a.table_words; j += gridDim.x * PREP_NT) ((uint32_t *)a.img)[j] = a.tables[j];
    }
}

// ---- the order of the sample -------------------------------------------------------------------------------------
// S = draws kept; slot i of the sample holds kept draw (i A + S / 3) mod S, A near S / golden ratio and coprime to S;
// the place of a draw needs A's inverse.
__device__ void sample_inverse(const ChainArgs &a)
{
    __shared__ uint32_t tot;
    if (threadIdx.x == 0) tot = 0;
    __syncthreads();
    const uint32_t S0 = sample_draws(a, a.scal->Nd), tiles = (S0 + DRAW_TILE - 1) / DRAW_TILE;
    uint32_t c = 0;
    for (uint32_t i = threadIdx.x; i < tiles; i += CLS_NT) c += a.kept[i];
    if (c) atomicAdd(&tot, c);
    __syncthreads();
    if (threadIdx.x != 0) return;
    const uint32_t S = tot;
    a.scal->S_enc = S;
    if (S <= 1) {
        a.scal->Ainv = 0;
        return;
    }
    uint32_t A = 1;
    if (S > 2) {
        A = (uint32_t)((double)S * 0.6180339887498949);
        A = min(max(A, 1u), S - 1);
        for (;; ++A) {  // S - 1 is coprime to S: the loop ends below S
            uint32_t x = A, y = S;
            while (x) {
                const uint32_t z = y % x;
                y = x;
                x = z;
            }
            if (y == 1) break;
        }
    }
    int64_t t = 0, nt = 1;
    uint32_t r = S, nr = A % S;
    while (nr) {
        const uint32_t q = r / nr, r2 = r - q * nr;
        const int64_t t2 = t - (int64_t)q * nt;
        t = nt; nt = t2; r = nr; nr = r2;
    }
    a.scal->Ainv = (uint32_t)(t < 0 ? t + S : t);
}

// blockIdx.y < T - 1: the distinct encodings into the buckets of tree y + 1; T - 1: the order of the sample
template <int KW, int KT>
__global__ void __launch_bounds__(CLS_NT) k_chain_classify_trees(ChainArgs a, uint32_t stride)
{
    extern __shared__ uint32_t blds[];
    if (a.scal->overflow) return;
    const int y = (int)blockIdx.y;
    if (y == a.T - 1) {
        if (blockIdx.x == 0) sample_inverse(a);
        return;
    }
    const uint32_t Nd = a.scal->Nd;
    if (blockIdx.x * (uint32_t)CLS_TILE >= Nd) return;
    const uint8_t *ecodes = (const uint8_t *)(a.img + offsets(a, Nd, 0).ecodes);
    const int t = y + 1, c0 = a.cb[t], D = a.cb[t + 1] - c0;
    classify<KT, 1>(tree_bufs(a, t), Nd, a.cap, a.wshift, stride, a.bstride, blds, [&](uint32_t i) {
        Elem<KT, 1> e;
        e.key = key_part<KW, KT>(key_of_row<KW>(ecodes, i, a.M, a.M == 4 * KW), c0, D);
        e.tail = i;
        return e;
    });
}

// ---- the samples into the image ----------------------------------------------------------------------------------
template <int KW, int NT>
__device__ void place_sample(const ChainArgs &a, uint32_t blk, uint32_t nblk)
{
    __shared__ uint32_t before, wave_n[DRAW_TILE / 64];
    const uint32_t Nd = a.scal->Nd, S = a.scal->S_enc, S0 = sample_draws(a, Nd), tiles = (S0 + DRAW_TILE - 1) / DRAW_TILE;
    const uint64_t Ainv = a.scal->Ainv, Bm = S / 3 % S;
    const Offsets o = offsets(a, Nd, S);
    const uint8_t *ecodes = (const uint8_t *)(a.img + o.ecodes), *rows = (const uint8_t *)(a.img + a.o_codes);
    uint32_t *out = (uint32_t *)(a.img + o.sample_enc), *pos = (uint32_t *)(a.img + o.sample_pos);
    uint8_t *out_rows = (uint8_t *)(a.img + o.sample_enc_codes), *pos_rows = (uint8_t *)(a.img + o.sample_pos_codes);
    const bool words = a.M == 4 * KW;
    const uint32_t lane = threadIdx.x & 63;
    for (uint32_t tile = blk; tile < tiles; tile += nblk) {
        __syncthreads();
        if (threadIdx.x == 0) before = 0;
        __syncthreads();
        uint32_t c = 0;
        for (uint32_t i = threadIdx.x; i < tile; i += NT) c += a.kept[i];
        if (c) atomicAdd(&before, c);
        for (uint32_t w = threadIdx.x >> 6; w < DRAW_TILE / 64; w += NT / 64) {
            const uint32_t s = tile * DRAW_TILE + w * 64 + lane;
            const uint64_t m = __ballot(s < S0 && (s == 0 || a.draw[s] != a.draw[s - 1]));
            if (lane == 0) wave_n[w] = (uint32_t)__popcll(m);
        }
        __syncthreads();
        for (uint32_t w = threadIdx.x >> 6; w < DRAW_TILE / 64; w += NT / 64) {
            const uint32_t s = tile * DRAW_TILE + w * 64 + lane;
            const bool keep = s < S0 && (s == 0 || a.draw[s] != a.draw[s - 1]);
            const uint64_t m = __ballot(keep);
            if (!keep) continue;
            uint64_t j = before + (uint32_t)__popcll(m & ((1ull << lane) - 1));
            for (uint32_t x = 0; x < w; ++x) j += wave_n[x];
            const uint64_t i = ((j + S - Bm) % S) * Ainv % S;
            const uint32_t e = a.draw[s];
            out[i] = e;
            row_of_key<KW>(out_rows, (int64_t)i, a.M, key_of_row<KW>(ecodes, e, a.M, words));
        }
    }
    // flat scan: one position from each of n_sample_pos strata
    const uint64_t n = (uint64_t)a.n_sample_pos, N = a.N;
    for (uint64_t i = (uint64_t)blk * NT + threadIdx.x; i < n; i += (uint64_t)nblk * NT) {
        const uint64_t s = (i * a.A_pos + a.B_pos) % n, lo = s * N / n, hi = (s + 1) * N / n;
        const uint64_t r = lo + mix64(a.seed ^ 0x5DEECE66Dull ^ s) % (hi - lo);
        pos[i] = (uint32_t)r;
        row_of_key<KW>(pos_rows, (int64_t)i, a.M, key_of_row<KW>(rows, (int64_t)r, a.M, words));
    }
}

// blockIdx.y < T - 1: sort of tree y + 1's buckets; T - 1: samples
template <int KW, int KT, int NT, uint32_t CAP>
__global__ void __launch_bounds__(NT) k_chain_sort_trees(ChainArgs a, uint32_t place_blocks)
{
    extern __shared__ uint32_t blds[];
    // Another workgroup of this launch may set the word at any time: one decision for all waves of a workgroup, or those
    // that go on would read LDS that those that left had yet to write.
    if (__syncthreads_or(a.scal->overflow != 0)) return;
    const int y = (int)blockIdx.y;
    if (y == a.T - 1) {
        if (blockIdx.x < place_blocks) place_sample<KW, NT>(a, blockIdx.x, place_blocks);
        return;
    }
    const uint32_t B = n_buckets(a.scal->Nd, a.cap, a.wshift), bucket = bucket_of_block(blockIdx.x, B);
    if ((blockIdx.x >> 3) >= (B + 7) / 8 || bucket >= B) return;
    bucket_sort<KT, 1, NT, CAP>(tree_bufs(a, y + 1), a.scal->Nd, a.bstride, bucket, 0, a.scal, blds);
}

// ---- a tree's leaves: number of every distinct encoding's, distinct sub-encodings --------------------------------
template <int KT, int NT>
__global__ void __launch_bounds__(NT) k_chain_leaves(ChainArgs a)
{
    if (a.scal->overflow) return;
    const int t = (int)blockIdx.y + 1;
    const uint32_t B = n_buckets(a.scal->Nd, a.cap, a.wshift);
    if (blockIdx.x >= B) return;
    const SortBufs s = tree_bufs(a, t);
    const BucketPlace pl = bucket_place<KT, NT>(s, B, blockIdx.x, 0);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.scal->U[t] = pl.tot;
    uint32_t *leaf = tree_leaf(a, t), *dk = tree_dk(a, t);
    bucket_walk<KT, 1, NT>(s, blockIdx.x, 0, pl, [&](uint32_t, const Elem<KT, 1> &x, bool head, uint32_t rank, bool, uint32_t) {
        leaf[x.tail] = rank - 1;
        if (head) key_store<KT>(dk + (int64_t)(rank - 1) * KT, x.key);
    });
}

template <int KT>
__global__ void __launch_bounds__(LVL_NT) k_chain_levels(ChainArgs a)
{
    if (a.scal->overflow) return;
    count_levels<KT>(a, (int)blockIdx.y, blockIdx.x);
}

// ---- the trees into the image ------------------------------------------------------------------------------------
// A workgroup writes the records and the nodes that start at its 4096 sub-encodings.  A node's number is the number of
// nodes of its kind and level up to it: the tiles before (summed here from their counts), the chunks of 64 before in the
// tile (LDS), the lanes before (ballot).
template <int KT> __device__ void write_levels(const ChainArgs &a, int t, uint32_t tile)
{
    __shared__ uint32_t cc[LVL_CH][CATS + 1], pre[CATS];
    __shared__ TreeOffsets o;
    __shared__ BuildScal scal;
    const uint32_t U = a.scal->U[t], lane = threadIdx.x & 63;
    if (tile * (uint32_t)LVL_TILE >= U) return;
    const int D = a.cb[t + 1] - a.cb[t];
    const Subs<KT> s = load_subs<KT>(tree_dk(a, t), tile, U, D);
    load_counts(a.scal, scal);
    if (threadIdx.x < CATS) pre[threadIdx.x] = 0;
    if (threadIdx.x == LVL_NT - 1) {
        int64_t off = offsets(a, scal.Nd, scal.S_enc).trees;
        for (int i = 0; i < t; ++i) place_tree(a, scal, i, off, [](int, int, int64_t) {});
        place_tree(a, scal, t, off, [&](int array, int l, int64_t at) {
            if (array == 1) o.rec = at;
            if (array == 2) o.icode[l] = at;
            if (array == 3) o.iparent[l] = at;
            if (array == 4) o.lcodes[l] = at;
            if (array == 5) o.lparent[l] = at;
            if (array == 6) o.lrow[l] = at;
        });
    }
    __syncthreads();
    {
        const uint32_t cat = threadIdx.x % CATS;
        uint32_t n = 0;
        for (uint32_t i = threadIdx.x / CATS; i < tile; i += LVL_NT / CATS) n += a.tile_cnt[((int64_t)t * a.lvl_tiles + i) * CATS + cat];
        if (n) atomicAdd(&pre[cat], n);
    }
#pragma unroll
    for (int q = 0; q < LVL_PER; ++q) {
        const uint32_t c = q * (LVL_NT / 64) + (threadIdx.x >> 6);
        const bool on = tile * LVL_TILE + c * 64 + lane < U;
        uint32_t mine = 0;
        for (int l = 1; l <= D; ++l) {
            const uint32_t ni = (uint32_t)__popcll(__ballot(on && is_internal(s.x[q], s.y[q], l, D))), nl = (uint32_t)__popcll(__ballot(on && is_leaf(s.x[q], s.y[q], l)));
            mine = (int)lane == l - 1 ? ni : (int)lane == ETF_MAX_M + l - 1 ? nl : mine;
        }
        if (lane < CATS) cc[c][lane] = mine;
    }
    __syncthreads();
    for (uint32_t cat = threadIdx.x >> 6; cat < CATS; cat += LVL_NT / 64) {
        static_assert(LVL_CH == 64, "a chunk per lane");
        const uint32_t n = cc[lane][cat];
        uint32_t x = n;
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(x, d);
            if ((int)lane >= d) x += y;
        }
        cc[lane][cat] = pre[cat] + x - n;
    }
    __syncthreads();
    const int dc = tree_depth_class(D), rwords = (dc < 4 ? 4 : dc) / 4;
    const uint64_t upto = ~0ull >> (63 - lane);
    uint8_t *rec = (uint8_t *)(a.img + o.rec);
#pragma unroll
    for (int q = 0; q < LVL_PER; ++q) {
        const uint32_t c = q * (LVL_NT / 64) + (threadIdx.x >> 6), u = tile * LVL_TILE + c * 64 + lane;
        const Key<KT> k = s.k[q];
        const int x = s.x[q], y = s.y[q];
        const bool on = u < U;
        if (on) key_write_front<KT>(rec + (int64_t)u * (4 * rwords), k >> (8 * (dc - D)), rwords);
        uint32_t parent = NO_PARENT;
        for (int l = 1; l <= D; ++l) {
            const bool in = on && is_internal(x, y, l, D), lf = on && is_leaf(x, y, l);
            const uint32_t upi = cc[c][l - 1] + (uint32_t)__popcll(__ballot(in) & upto);
            const uint32_t upl = cc[c][ETF_MAX_M + l - 1] + (uint32_t)__popcll(__ballot(lf) & upto);
            if (in) {
                ((uint8_t *)(a.img + o.icode[l - 1]))[upi - 1] = key_chunk<KT>(k, l - 1);
                ((uint32_t *)(a.img + o.iparent[l - 1]))[upi - 1] = parent;
            }
            if (lf) {
                const int words = (D - l + 1 + 3) / 4;
                key_write_front<KT>((uint8_t *)(a.img + o.lcodes[l - 1]) + (int64_t)(upl - 1) * (4 * words), k << (8 * (l - 1)), words);
                ((uint32_t *)(a.img + o.lparent[l - 1]))[upl - 1] = parent;
                ((uint32_t *)(a.img + o.lrow[l - 1]))[upl - 1] = u;
            }
            parent = upi - 1;  // u's own group, or the last one that started before u
        }
    }
}

// leaf numbers and tree 0's chunks of every distinct encoding
template <int KW> __device__ void write_encodings(const ChainArgs &a, uint32_t blk)
{
    __shared__ int64_t leaf_of[ETF_MAX_M];
    __shared__ BuildScal scal;
    const uint32_t Nd = a.scal->Nd;
    if (blk * (uint32_t)LVL_TILE >= Nd) return;
    load_counts(a.scal, scal);
    const Offsets o = offsets(a, Nd, scal.S_enc);
    if (a.T > 1 && threadIdx.x == 0) {
        int64_t off = o.trees;
        for (int t = 0; t < a.T; ++t)
            place_tree(a, scal, t, off, [&](int array, int, int64_t at) {
                if (array == 0) leaf_of[t] = at;
            });
    }
    __syncthreads();
    const int D0 = a.cb[1], dc = tree_depth_class(D0), words = a.rstride0 / 4;
    const uint8_t *ecodes = (const uint8_t *)(a.img + o.ecodes);
    uint8_t *rec0 = (uint8_t *)(a.img + o.rec0);
    for (uint32_t e = blk * LVL_TILE + threadIdx.x; e < min((blk + 1) * (uint32_t)LVL_TILE, Nd); e += LVL_NT) {
        const Key<KW> k = key_part<KW, KW>(key_of_row<KW>(ecodes, e, a.M, a.M == 4 * KW), 0, D0);
        key_write_front<KW>(rec0 + (int64_t)e * a.rstride0, k >> (8 * (dc - D0)), words);
        if (a.T > 1)
            for (int t = 0; t < a.T; ++t) ((uint32_t *)(a.img + leaf_of[t]))[e] = tree_leaf(a, t)[e];
    }
}

// blockIdx.y < T: levels and records of tree y; T: the encodings' leaf numbers and records
template <int KW, int KT>
__global__ void __launch_bounds__(LVL_NT) k_chain_write(ChainArgs a)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < sizeof(BuildScal) / 4)
        ((uint32_t *)a.scal_host)[threadIdx.x] = ((const uint32_t *)a.scal)[threadIdx.x];
    if (a.scal->overflow) return;
    if ((int)blockIdx.y < a.T) write_levels<KT>(a, (int)blockIdx.y, blockIdx.x);
    else write_encodings<KW>(a, blockIdx.x);
}
