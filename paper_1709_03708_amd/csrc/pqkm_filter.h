// Assignment scans through a lower bound (Eq. 5 over Eq. 3, exact results).
//
// The LDS-tiled scans of pqkm_kernels.h form every fp32 distance: M four-byte look-ups and M - 1 adds per code and
// center, and the LDS and the vector units are both near their limit doing so.  Nearly all of that work goes into
// centers that are far from being the nearest.  Here the scan sums one-byte lower bounds of the table entries instead,
// four centers per 32-bit register, and only the few centers whose bound does not exceed the code's best distance so far
// get their fp32 distance, formed from the caller's tables in the order of Eq. 3.  The result is that of the plain
// scan, bit for bit: a center that is skipped has an fp32 distance strictly above one that was formed.
//
// The bound.  With lo_m = the smallest finite entry of A^m, U = (A^m[x][c] - lo_m) * inv is an entry in units, and
// q = min(31, floor(U (1 - 2^-20))) <= U.  Let s be the fp32 distance of (code, center) and b the code's best so far.
// s <= b implies sum_m A <= b + err with err = (M + 2) 2^-23 sum_m max|A^m| (rounding of the fp32 sum, of lo_m and of
// the differences), so sum_m q <= (b - sum_m lo_m + err) inv; the threshold is that, rounded up.  A NaN or +inf entry
// takes q = 31: a distance that contains one is never selected, so skipping it is right.  A -inf entry, tables without
// spread, or differences that overflow set inv = 0: every bound is 0 and passes, which is correct and then handled as
// below.  inv = 31 / min(largest difference, 1.75 times the mean one): entries beyond are
// capped, which only loosens the bound (between 1.5 and 2 the fewest centers pass on codes of clustered data).
//
// Where the bound selects too little (ties everywhere, tables without spread) forming the fp32 distances one by one
// would be slower than the plain scan.  A workgroup counts the candidates it has formed and gives up when what is left would
// cost it more than the plain scan of everything (filter_budget); its codes are then left to the plain scan that is launched
// behind this one and ends at once where nothing was left to it.
#pragma once
#include "pqkm_kernels.h"

namespace pqkm {

constexpr int FILTER_Q = 31;              // largest bound of an entry (M = 16, 32: FILTER_Q_WIDE)
constexpr int FILTER_Q_WIDE = 63;
constexpr int FILTER_TK = 64;             // centers per tile: a row of one subcode is 64 bytes
constexpr uint32_t FILTER_PLANE = 16384;  // bytes per (tile, subspace): 256 subcodes x 64 centers
constexpr int FILTER_QUEUE = 128;         // candidate entries a wave can hold (drained from 64 on)

// Clocks of a compute unit per code: the plain scan of 64 centers, this one's, and a candidate, from the times beside the
// kernels below.  A candidate is M table entries through the L2 at 5 clocks each; at M = 4 its entry's code, key and center
// count as well (27 clocks at N = 1e6, K = 20000).  first, later, share: candidates per code that a first and a later
// iteration may take before their rate counts, at least that share of the plain scan.  Codes start from a bound that the
// first tiles improve: where the scan gains, clustered codes and Gaussian codewords take 2 to 5 candidates in the first
// four tiles at M = 4, 3 to 7 at M = 8, 3 to 9 at M = 16 and 6 to 12 at M = 32, and then 0.1 per tile and less; with
// distances that are small integers it is up to one per tile throughout.
template <int M> struct FilterCost;
template <> struct FilterCost<4> { static constexpr float plain = 5.5f, scan = 1.7f, candidate = 30.0f, first = 6.0f, later = 2.0f, share = 0.375f; };
template <> struct FilterCost<8> { static constexpr float plain = 12.0f, scan = 4.5f, candidate = 40.0f, first = 10.0f, later = 6.0f, share = 0.25f; };
template <> struct FilterCost<16> { static constexpr float plain = 39.0f, scan = 22.0f, candidate = 80.0f, first = 10.0f, later = 7.0f, share = 0.3f; };
template <> struct FilterCost<32> { static constexpr float plain = 64.0f, scan = 37.0f, candidate = 160.0f, first = 12.0f, later = 8.0f, share = 0.3f; };

// Candidates per code that are worth going on with after t of T tiles.  Giving up costs the plain scan of all T tiles; going on,
// the T - t that are left at the rate r of candidates per tile seen so far, (scan + r candidate) (T - t).  The two are equal at
// r = (plain T / (T - t) - scan) / candidate.  On top of that what is free.
template <int M>
__device__ __forceinline__ float filter_budget(int t, int T, bool later)
{
    typedef FilterCost<M> Cost;
    const float rate = (Cost::plain * (float)T / (float)(T - t) - Cost::scan) * (1.0f / Cost::candidate);
    return __builtin_fmaxf(later ? Cost::later : Cost::first, Cost::share * Cost::plain / Cost::candidate * (float)T) + (float)t * rate;
}

// statistics of the tables, FILTER_PARTS blocks per subspace; st[m * FILTER_PARTS + part]
constexpr int FILTER_PARTS = 8;
struct FilterStat { float lo, hi, mean, absmax; };       // finite entries; lo = -inf if there is a -inf entry

__global__ __launch_bounds__(1024) void filter_stats_kernel(const float* __restrict__ tables, FilterStat* __restrict__ st,
                                                            const uint32_t* __restrict__ only_if = nullptr)
{
    if (only_if && *only_if == 0u) return;
    __shared__ float lo_s[16], hi_s[16], sum_s[16];
    constexpr int PART = L * L / FILTER_PARTS;
    const float* part = tables + (size_t)blockIdx.x * PART;
    const float4* t = reinterpret_cast<const float4*>(part);
    const bool aligned = ((uintptr_t)tables & 15) == 0;
    float lo = INFINITY, hi = -INFINITY, sum = 0.0f;
    auto take = [&](float v) {
        if (v == -INFINITY) lo = v;
        if (__builtin_fabsf(v) < INFINITY) {
            lo = v < lo ? v : lo;
            hi = v > hi ? v : hi;
            sum += v;
        }
    };
    if (aligned) {
#pragma unroll
        for (int i = threadIdx.x; i < PART / 4; i += 1024) {
            const float4 v = t[i];
            take(v.x); take(v.y); take(v.z); take(v.w);
        }
    } else {
        for (int i = threadIdx.x; i < PART; i += 1024) take(part[i]);
    }
#pragma unroll
    for (int off = 32; off; off >>= 1) {
        lo = __builtin_fminf(lo, __shfl_xor(lo, off));
        hi = __builtin_fmaxf(hi, __shfl_xor(hi, off));
        sum += __shfl_xor(sum, off);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { lo_s[w] = lo; hi_s[w] = hi; sum_s[w] = sum; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < 16; ++i) {
            lo = __builtin_fminf(lo, lo_s[i]);
            hi = __builtin_fmaxf(hi, hi_s[i]);
            sum += sum_s[i];
        }
        st[blockIdx.x] = FilterStat{lo, hi, sum / (float)PART, __builtin_fmaxf(__builtin_fabsf(lo), __builtin_fabsf(hi))};
    }
}

// the smallest finite entry of A^m (-inf if there is a -inf entry)
__device__ __forceinline__ float filter_low(const FilterStat* __restrict__ st, int m)
{
    float lo = st[m * FILTER_PARTS].lo;
#pragma unroll
    for (int i = 1; i < FILTER_PARTS; ++i) lo = __builtin_fminf(lo, st[m * FILTER_PARTS + i].lo);
    return lo;
}

// what the scan needs of the statistics: units = (value - base) * inv + slack
struct FilterScale { float inv, base, slack; };

template <int M>
__device__ __forceinline__ FilterScale filter_scale(const FilterStat* __restrict__ st)
{
    float span = 0.0f, mean = 0.0f, base = 0.0f, absmax = 0.0f;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        FilterStat s = st[m * FILTER_PARTS];
#pragma unroll
        for (int i = 1; i < FILTER_PARTS; ++i) {
            const FilterStat o = st[m * FILTER_PARTS + i];
            s.lo = __builtin_fminf(s.lo, o.lo);
            s.hi = __builtin_fmaxf(s.hi, o.hi);
            s.mean += o.mean;
            s.absmax = __builtin_fmaxf(s.absmax, o.absmax);
        }
        const float d = s.hi - s.lo;
        span = (d > span || !(d == d)) ? d : span;
        mean += s.mean / (float)FILTER_PARTS - s.lo;
        base += s.lo;
        absmax += s.absmax;
    }
    float cap = 1.75f * (mean / (float)M);
    cap = span < cap ? span : cap;
    FilterScale f;
    f.inv = (float)(M >= 16 ? FILTER_Q_WIDE : FILTER_Q) / cap;
    // no spread, -inf or NaN anywhere, or an inverse out of range: everything passes
    if (!(span > 0.0f && span < INFINITY) || !(cap > 0.0f) || !(f.inv > 0.0f && f.inv < 1e30f) || !(absmax < 1e30f)) f.inv = 0.0f;
    f.base = f.inv > 0.0f ? base : 0.0f;
    f.slack = f.inv > 0.0f ? 0.01f + (float)(M + 2) * 0x1p-23f * absmax * f.inv : 0.0f;
    return f;
}

__device__ __forceinline__ uint32_t filter_quantise(float a, float lo, float inv, int most)
{
    const float u = (a - lo) * inv * (1.0f - 0x1p-20f);
    return u < (float)most ? (uint32_t)(u > 0.0f ? u : 0.0f) : (uint32_t)most;              // NaN and +inf: the cap
}

// largest sum of bounds a center may have, at most `tmax` (which passes everything); best = NaN or +inf: tmax
__device__ __forceinline__ uint32_t filter_threshold(float best, const FilterScale& f, uint32_t tmax)
{
    const float u = (best - f.base) * f.inv * (1.0f + 0x1p-18f) + f.slack;
    if (!(f.inv > 0.0f) || !(best < INFINITY)) return tmax;
    return u < (float)tmax ? (uint32_t)(u > 0.0f ? u : 0.0f) : tmax;
}

// img[tile][m][x][64 centers]: block (tile, m, quarter of the subcodes), 256 threads of 16 bytes each.  Centers past K
// take the cap; the scan drops them by their index.
template <int M>
__global__ __launch_bounds__(256) void filter_image_kernel(const uint8_t* __restrict__ centers, int K,
                                                            const float* __restrict__ tables,
                                                            const FilterStat* __restrict__ st, uint4* __restrict__ img,
                                                            uint8_t* __restrict__ copy, FilterScale* __restrict__ scale,
                                                            uint32_t* __restrict__ gave_up)
{
    static_assert(M < 16, "M = 16, 32: filter_wide_image_kernel");
    __shared__ uint32_t sub[FILTER_TK];
    const int tile = (int)(blockIdx.x / (4 * M)), m = (int)(blockIdx.x / 4 % M), part = (int)(blockIdx.x % 4);
    const FilterScale sc = filter_scale<M>(st);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *scale = sc;                                                 // for the scan
        *gave_up = 0u;
    }
    const float inv = sc.inv, lo = filter_low(st, m);
    if (threadIdx.x < FILTER_TK) {
        const int64_t k = (int64_t)tile * FILTER_TK + threadIdx.x;
        sub[threadIdx.x] = k < K ? centers[k * M + m] : 256u;
        if (copy && part == 0 && k < K) copy[k * M + m] = centers[k * M + m];       // for the next iteration's comparison
    }
    __syncthreads();
    const int x = part * 64 + (threadIdx.x >> 2), p = threadIdx.x & 3;
    const float* row = tables + ((size_t)m * L + x) * L;
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t c = sub[p * 16 + i];
        v[i] = c < 256u ? row[c] : INFINITY;
    }
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i >> 2] |= filter_quantise(v[i], lo, inv, FILTER_Q) << (8 * (i & 3));
    img[((size_t)tile * M + m) * 1024 + part * 256 + threadIdx.x] = make_uint4(w[0], w[1], w[2], w[3]);
}

// M = 16, 32: the tables as bytes first, [m][x][256], so that the images read a quarter of what they read of the tables (K = 10000,
// M = 32: 1.3 GB through the L2 for images of 82 MB, 201 us; 15 for the bytes and 54 for the images from their rows in LDS).
template <int M>
__global__ __launch_bounds__(256) void filter_bytes_kernel(const float* __restrict__ tables, const FilterStat* __restrict__ st,
                                                            uint32_t* __restrict__ bytes, FilterScale* __restrict__ scale,
                                                            uint32_t* __restrict__ gave_up, const uint32_t* __restrict__ only_if)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *gave_up = 0u;                     // also where the scan has nothing to do
    if (only_if && *only_if == 0u) return;
    const FilterScale sc = filter_scale<M>(st);
    if (blockIdx.x == 0 && threadIdx.x == 0) *scale = sc;                        // for the scan
    const int m = (int)blockIdx.x / 16;
    const float lo = filter_low(st, m);
    const size_t first = (size_t)blockIdx.x * 4096;                              // 16 rows
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const size_t at = first + i * 1024 + threadIdx.x * 4;
        uint32_t w = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) w |= filter_quantise(tables[at + j], lo, sc.inv, FILTER_Q_WIDE) << (8 * j);
        bytes[at / 4] = w;
    }
}

// img[tile][m / 4][x][m % 4][64 centers], the phases of four subspaces: block (tile, m, quarter of the subcodes) with its 64 rows of bytes in
// LDS, 16 bytes per thread.  Centers past K take the cap; the scan drops them by their index.
template <int M>
__global__ __launch_bounds__(256) void filter_wide_image_kernel(const uint8_t* __restrict__ centers, int K,
                                                                 const uint4* __restrict__ bytes, uint4* __restrict__ img,
                                                                 const uint32_t* __restrict__ only_if)
{
    __shared__ uint4 rows[64 * 16];
    __shared__ uint32_t sub[FILTER_TK];
    if (only_if && *only_if == 0u) return;
    const int tile = (int)(blockIdx.x / (4 * M)), m = (int)(blockIdx.x / 4 % M), part = (int)(blockIdx.x % 4);
    const uint4* from = bytes + ((size_t)m * L + part * 64) * 16;
#pragma unroll
    for (int i = 0; i < 4; ++i) rows[i * 256 + threadIdx.x] = from[i * 256 + threadIdx.x];
    if (threadIdx.x < FILTER_TK) {
        const int64_t k = (int64_t)tile * FILTER_TK + threadIdx.x;
        sub[threadIdx.x] = k < K ? centers[k * M + m] : 256u;
    }
    __syncthreads();
    const int xr = threadIdx.x >> 2, p = threadIdx.x & 3;
    const uint8_t* row = reinterpret_cast<const uint8_t*>(rows) + xr * 256;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t c = sub[p * 16 + i];
        w[i >> 2] |= (c < 256u ? (uint32_t)row[c] : (uint32_t)FILTER_Q_WIDE) << (8 * (i & 3));
    }
    img[((size_t)tile * (M / 4) + m / 4) * 4096 + (size_t)(part * 64 + xr) * 16 + (m % 4) * 4 + p] = make_uint4(w[0], w[1], w[2], w[3]);
}

// For every pair of neighbouring subspaces and every pair of subcodes some center that has both (which one does not
// matter): codes of clustered data nearly always share a pair with a center close to them.
template <int M, int PAIRS = M / 2>
__global__ __launch_bounds__(256) void filter_pairs_kernel(const uint8_t* __restrict__ centers, int K,
                                                           uint32_t* __restrict__ pairs,
                                                           const uint32_t* __restrict__ only_if = nullptr)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= K || (only_if && *only_if == 0u)) return;
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        const uint32_t c = centers[(size_t)k * M + 2 * p] | ((uint32_t)centers[(size_t)k * M + 2 * p + 1] << 8);
        pairs[(size_t)p * 65536 + c] = (uint32_t)k;
    }
}

// (distance, center) as one integer whose order is "smaller distance, then lower index"; -0 counts as +0
__device__ __forceinline__ unsigned long long filter_key(float s, uint32_t k)
{
    const float z = s + 0.0f;
    const uint32_t u = __builtin_bit_cast(uint32_t, z);
    const uint32_t o = u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
    return ((unsigned long long)o << 32) | k;
}
__device__ __forceinline__ float filter_key_distance(unsigned long long key)
{
    const uint32_t o = (uint32_t)(key >> 32);
    return __builtin_bit_cast(float, o ^ ((o >> 31) ? 0x80000000u : 0xffffffffu));
}
constexpr unsigned long long FILTER_NONE = ~0ull;        // no center selected yet (GAVE_UP: left to the plain scan)

struct FilterIn {
    const uint4* img;                // byte tiles
    const float* tables;
    const uint8_t* centers;          // 4-byte aligned
    const FilterScale* scale;
    unsigned long long* state;       // one key per code position of the launch
    int K, ntiles;                   // ntiles = ceil(K / 64)
    const uint8_t* before;           // the centers of the iteration whose keys `state` holds (seeded == 2)
    const uint32_t* pairs;           // seeded == 3: [M / 2][65536], a center with these two subcodes, or >= K
    int seeded;                      // 0: nothing known; 1: assign[] holds a center for every code (of the iteration before);
                                     // 2: so does `state`; 3: `pairs` names candidates
    uint32_t* gave_up;               // workgroups of this stretch of codes that gave up
    int launched;                    // workgroups of it in earlier launches: if most of those gave up, so do these
};

// a code of the regrouped array (M = 4: code, origin; M = 8: code, code, origin, -) and a center, packed in words
template <int M> struct FilterCode;
template <> struct FilterCode<4> {
    typedef uint2 Raw;
    uint32_t w[1], origin;
    __device__ __forceinline__ explicit FilterCode(uint2 v) : w{v.x}, origin(v.y) {}
    __device__ __forceinline__ FilterCode() {}
};
template <> struct FilterCode<8> {
    typedef uint4 Raw;
    uint32_t w[2], origin;
    __device__ __forceinline__ explicit FilterCode(uint4 v) : w{v.x, v.y}, origin(v.z) {}
    __device__ __forceinline__ FilterCode() {}
};
template <int W> struct FilterWords { uint32_t w[W]; };

// the fp32 distance of Eq. 3
template <int M>
__device__ __forceinline__ float filter_distance(const float* __restrict__ tables, const uint32_t (&x)[M / 4],
                                                 const FilterWords<M / 4>& c)
{
    float a[M];
#pragma unroll
    for (int m = 0; m < M; ++m)
        a[m] = tables[((uint32_t)m << 16) | (((x[m / 4] >> (8 * (m % 4))) & 255u) << 8) | ((c.w[m / 4] >> (8 * (m % 4))) & 255u)];
    float s = a[0];
#pragma unroll
    for (int m = 1; m < M; ++m) s = s + a[m];
    return s;
}

// ---------------------------------------------------------------------------------------------
// M = 4, 8: regrouped codes and two-lane slots of assign_scan4h_kernel and assign_scan8q_kernel, whose 64-byte rows of 16
// fp32 centers are here rows of 64 one-byte centers, with the same conflict-free reads.  Per code and tile of 64 centers a
// lane reads 2 x 16 bytes per subspace = 32 centers and adds the bounds of four centers per instruction (three-operand
// adds; at most M * 31 = 248, no byte carries into its neighbour).  A byte per code holds what the sum must stay below:
// M = 4 adds 127 - threshold (the sum of both is at most 252), M = 8 averages with 254 - threshold, rounding up
// (v_lerp_u8); either way the high bit of a byte ends up clear exactly when the center passes.  128 or 255 in its place
// lets nothing pass (the holes of the regrouped array).  The high bits of two codes are and'ed into one test per wave;
// lanes with a clear one append (mask of 32 centers, code, tile) to a queue of their wave in LDS, and 64 entries are
// worked off at a time, one lane each: subcodes of the center, M table entries through the L2, an atomic minimum of
// (distance, index) on the code's key in global memory, the new threshold to LDS.  Thresholds are read four codes at a
// time when a tile begins.  Before the first tile every code needs a bound: the distance to its center of the previous
// iteration, where there is one; in a first iteration the distance to the closest of a few centers that share two neighbouring subcodes
// with it, or else to the center with the smallest sum of bounds in the first tile.
// A tile is 64 KB at M = 4: two buffers, the next tile's loads straight into LDS run beside the scan.  At M = 8 it is
// 128 KB, one buffer, loaded between two barriers (about 3000 clocks for 14000 of scan with 4096 codes).
//
// Bound by vector issue and LDS reads together (a wave takes about 175 clocks of its SIMD per 32 codes and tile at
// M = 4, of which the 8 reads are 64), and with few centers by the candidates: a table entry through the L2 costs a
// compute unit about 5 clocks, a candidate M of them.
// Measured, plain scan -> this: M = 4, N = 2e6, K = 1e5: 26.5 -> 8.7 ms (2.3e13 code-center pairs/s); N = 3e6,
// K = 2500: 1.27 -> 1.05 ms in a first iteration, 0.69 ms in later ones.  M = 8, N = 1e7,
// K = 1e4: 30.2 -> 18.0 ms in a first iteration, 13.0 and 11.5 ms in later ones.
// ---------------------------------------------------------------------------------------------
template <int V> struct IntC { static constexpr int value = V; };

typedef unsigned short v2us __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(v2us, a), __builtin_bit_cast(v2us, b)));
}

template <int M, int R, int THREADS, int DEPTH, bool BUCKET>
__global__ __launch_bounds__(THREADS) void assign_filter_kernel(int64_t N, const typename FilterCode<M>::Raw* __restrict__ gco,
                                                             FilterIn f, int32_t* __restrict__ assign,
                                                             float* __restrict__ dist, RankOut ro, BucketOut bo)
{
    constexpr int SLOTS = THREADS / 2, C = SLOTS * R, TW = R / 4, W = M / 4;
    constexpr int CHUNKS = (int)FILTER_PLANE / (THREADS * 16);              // loads per plane
    constexpr int BUFFERS = M == 4 ? 2 : 1;
    constexpr uint32_t STRIDE = BUFFERS * FILTER_PLANE;                     // bytes between two subspaces in LDS
    constexpr uint32_t ALL = M == 4 ? 127u : 254u, DEAD = ALL + 1u;         // what passes everything; the byte of a hole
    constexpr uint32_t HI = 0x80808080u;
    static_assert(R % 4 == 0, "thresholds are read as words of four codes");
    static_assert(M * FILTER_Q < 255, "a sum of bounds fits a byte");
    __shared__ float4 tile[TILE_F4];
    __shared__ uint32_t thr_s[SLOTS * TW];
    __shared__ uint2 queue_s[THREADS / 64][FILTER_QUEUE];
    __shared__ uint32_t spent_s, quit_s, bail_s[2];
    __shared__ uint32_t gcnt[BUCKET ? 256 : 1], gbase[BUCKET ? 256 : 1];
    const char* tb = reinterpret_cast<const char*>(tile);
    uint8_t* thr_b = reinterpret_cast<uint8_t*>(thr_s);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = tid & 1, c = tid >> 1;
    const uint32_t hq = ((uint32_t)(c & 1) << 5) | ((uint32_t)q << 4);
    const int64_t base = (int64_t)blockIdx.x * C;
    const uint32_t low15 = 0x7fffu;
    uint2* queue = queue_s[wave];

    // plane m of buffer h at byte m * STRIDE + h * 16384
    const uint64_t ip = reinterpret_cast<uint64_t>(f.img);
    constexpr uint32_t TILE = M * FILTER_PLANE;
    const v4i rs_img = {(int)(uint32_t)ip, (int)(uint32_t)(ip >> 32), (int)((uint32_t)f.ntiles * TILE), 0x00020000};
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)tile;
    const uint32_t wave_off = (uint32_t)wave * 1024u, lane_off = (uint32_t)tid * 16u;
    auto fetch = [&](int t, int h, int j) {
        const uint32_t m = (uint32_t)(j / CHUNKS), part = (uint32_t)(j % CHUNKS) * (THREADS * 16);
        buffer_to_lds16(lds0 + m * STRIDE + (uint32_t)h * FILTER_PLANE + part + wave_off, rs_img, lane_off,
                        (uint32_t)t * TILE + m * FILTER_PLANE + part);
    };
#pragma unroll
    for (int j = 0; j < M * CHUNKS; ++j) fetch(0, 0, j);

    const FilterScale sc = *f.scale;
    const FilterWords<W>* cen = reinterpret_cast<const FilterWords<W>*>(f.centers);
    static_assert(C % GAVE_UP_STEP == 0, "the plain scan looks at one key per step");
    auto give_up = [&]() {
        wait_vector_loads();                     // nothing may land in LDS after the workgroup has ended
        for (int i = tid; i < C; i += THREADS)
            if (base + i < N) f.state[base + i] = GAVE_UP;
        if (tid == 0) atomicAdd(f.gave_up, 1u);
    };
    if (tid == 0) {
        spent_s = 0u;
        // tables that the bounds say nothing about
        const uint32_t left = __hip_atomic_load(f.gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        quit_s = !(sc.inv > 0.0f) || (f.launched > 0 && 2u * left > (uint32_t)f.launched) ? 1u : 0u;
    }
    if (tid < 2) bail_s[tid] = 0u;
    __syncthreads();
    if (quit_s) {
        give_up();
        return;
    }

    // keys and thresholds of the workgroup's codes; the loads of a few codes travel together
    constexpr int SB = M == 8 ? 2 : (R / 2) % 4 == 0 ? 4 : (R / 2) % 3 == 0 ? 3 : 2;
    static_assert((R / 2) % SB == 0, "whole batches");
#pragma unroll 1
    for (int i0 = 0; i0 < R / 2; i0 += SB) {
        FilterCode<M> g[SB];
        uint32_t k[SB];
        float s[SB];
        unsigned long long old[SB];
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int64_t n = base + (i0 + i) * THREADS + tid, nc = n < N ? n : N - 1;
            g[i] = FilterCode<M>(gco[nc]);
            if (n >= N) g[i].origin = ORIGIN_NONE;
            old[i] = f.seeded == 2 ? f.state[nc] : FILTER_NONE;
            k[i] = (uint32_t)old[i];
        }
        if (f.seeded == 3) {
            // the closest of the centers that share a pair of subcodes with the code
            uint32_t cand[SB][M / 2];
#pragma unroll
            for (int i = 0; i < SB; ++i)
#pragma unroll
                for (int p = 0; p < M / 2; ++p)
                    cand[i][p] = f.pairs[p * 65536 + ((g[i].w[p / 2] >> (16 * (p % 2))) & 0xffffu)];
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                s[i] = INFINITY;
                k[i] = 0xffffffffu;
#pragma unroll
                for (int p = 0; p < M / 2; ++p) {
                    const uint32_t kk = cand[i][p];
                    if (kk < (uint32_t)f.K && kk != k[i]) {
                        const float d = filter_distance<M>(f.tables, g[i].w, cen[kk]);
                        if (d < s[i] || (d == s[i] && kk < k[i])) { s[i] = d; k[i] = kk; }
                    }
                }
            }
        } else if (f.seeded) {
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                if (f.seeded == 1 || old[i] == GAVE_UP) k[i] = (uint32_t)assign[g[i].origin == ORIGIN_NONE ? 0u : g[i].origin];
                k[i] = k[i] < (uint32_t)f.K ? k[i] : 0u;             // any center will do
            }
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                // an unchanged center is as far as it was; table entries are fetched for the others only
                const FilterWords<W> now = cen[k[i]];
                s[i] = filter_key_distance(old[i]);
                bool same = f.seeded == 2 && old[i] != FILTER_NONE && old[i] != GAVE_UP;
                if (same) {
                    const FilterWords<W> was = reinterpret_cast<const FilterWords<W>*>(f.before)[k[i]];
#pragma unroll
                    for (int w = 0; w < W; ++w) same = same && was.w[w] == now.w[w];
                }
                if (!same) s[i] = filter_distance<M>(f.tables, g[i].w, now);
            }
        }
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int jj = (i0 + i) * THREADS + tid;
            unsigned long long key = FILTER_NONE;
            uint32_t t = g[i].origin == ORIGIN_NONE ? DEAD : 0u;
            if (f.seeded && g[i].origin != ORIGIN_NONE && s[i] < INFINITY) {
                key = filter_key(s[i], k[i]);
                t = ALL - filter_threshold(s[i], sc, ALL);
            }
            if (base + jj < N) f.state[base + jj] = key;
            thr_b[(jj % SLOTS) * R + jj / SLOTS] = (uint8_t)t;
        }
    }

    // packed row offsets: subspace m < M/2 in the low 15 bits, m + M/2 (64 KB higher) from bit 15 up
    uint32_t fld[R][M / 2];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int64_t n = base + (int64_t)r * SLOTS + c;
        if (n >= N) n = N - 1;
        const FilterCode<M> g(gco[n]);
#pragma unroll
        for (int m = 0; m < M / 2; ++m) {
            const int m2 = m + M / 2;
            const uint32_t xa = (g.w[m / 4] >> (8 * (m % 4))) & 255u, xb = (g.w[m2 / 4] >> (8 * (m2 % 4))) & 255u;
            fld[r][m] = ((xa << 6) | hq) | ((((xb << 6) | hq) + 65536u) << 15);
        }
    }
    auto row_of = [&](int r, int m) -> uint32_t {
        return m < M / 2 ? unpack_low15(low15, fld[r][m]) : unpack_high17(fld[r][m - M / 2]);
    };

    int qn = 0;                                  // entries in the wave's queue (the same in all lanes)
    // candidates that the workgroup may have formed up to the tile at hand
    const bool later = f.seeded == 1 || f.seeded == 2;
    float allowed = filter_budget<M>(0, f.ntiles, later) * (float)C;

    // up to 64 entries, one lane each
    auto drain = [&]() __attribute__((always_inline)) {
        if ((float)__builtin_amdgcn_readfirstlane(spent_s) > allowed) {
            quit_s = 1u;
            qn = 0;
            return;
        }
        const int cnt = qn < 64 ? qn : 64;
        qn -= cnt;
        __builtin_amdgcn_wave_barrier();
        const uint2 e = queue[qn + (lane < cnt ? lane : 0)];
        __builtin_amdgcn_wave_barrier();
        uint32_t mask = lane < cnt ? e.x : 0u;
        const uint32_t r = e.y & 31u, sl = (e.y >> 5) & 31u, eq = (e.y >> 10) & 1u, t = e.y >> 11;
        const int slot = wave * 32 + (int)sl;
        const int64_t n = base + (int64_t)r * SLOTS + slot;
        const uint32_t piece = 2u * (sl & 1u) + eq;
        const FilterCode<M> x(gco[n]);           // only positions below N ever pass
        // the center the key names already (the bound a code starts with is often its answer) needs no second look
        const unsigned long long known = __hip_atomic_load(&f.state[n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        {
            const uint32_t in = (uint32_t)known - t * FILTER_TK;           // its place in this tile, if it is here
            if (known != FILTER_NONE && in < (uint32_t)FILTER_TK && ((in >> 4) & ~2u) == (piece & ~2u)) {
                const uint32_t j = (((in >> 4) == piece) ? 0u : 4u) + ((in >> 2) & 3u);
                mask &= ~(1u << (8u * (in & 3u) + 7u - j));
            }
        }
        float sb = INFINITY;
        uint32_t kb = 0xffffffffu;
        uint32_t formed = 0u;
        while (true) {
            const uint64_t who = __ballot(mask != 0u);
            if (!who) break;
            formed += (uint32_t)__builtin_popcountll(who);
            if (mask) {
                const uint32_t bit = (uint32_t)__builtin_ctz(mask), j = 7u - (bit & 7u);
                mask &= mask - 1u;
                const uint32_t k = t * FILTER_TK + 16u * (piece ^ ((j >> 2) << 1)) + 4u * (j & 3u) + (bit >> 3);
                if (k < (uint32_t)f.K) {
                    const float s = filter_distance<M>(f.tables, x.w, cen[k]);
                    if (s < INFINITY && (s < sb || (s == sb && k < kb))) { sb = s; kb = k; }
                }
            }
        }
        if (kb != 0xffffffffu) {                 // some distance below +inf
            atomicMin(&f.state[n], filter_key(sb, kb));
            const uint32_t nt = ALL - filter_threshold(sb, sc, ALL);
            uint8_t* p = thr_b + slot * R + r;
            if (nt > *p) *p = (uint8_t)nt;
        }
        if (lane == 0) atomicAdd(&spent_s, formed);
    };
    // The lanes with a clear high bit in what they hold of code r0 (a0; n0 is the and of its registers) or r1 append
    // their 32 centers: bit 8 b + 7 - j for byte b of register j.  A lane with both appends twice.
    auto push = [&](const uint32_t (&a0)[8], const uint32_t (&a1)[8], uint32_t n0, uint32_t n1, int r0, int r1, int t)
        __attribute__((always_inline)) {
        bool p0 = (n0 & HI) != HI, p1 = (n1 & HI) != HI;
#pragma unroll 1
        while (true) {
            const uint64_t who = __ballot(p0 || p1);
            if (!who) break;
            uint32_t m = 0u;
#pragma unroll
            for (int j = 7; j >= 0; --j) {
                const uint32_t v = p0 ? a0[j] : a1[j];
                m = j == 7 ? v : (v & HI) | ((m >> 1) & ~HI);
            }
            m = ~m;
            const int at = qn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
            if (p0 || p1)
                queue[at] = make_uint2(m, (uint32_t)(p0 ? r0 : r1) | ((uint32_t)(lane >> 1) << 5) | ((uint32_t)q << 10) | ((uint32_t)t << 11));
            p1 = p0 && p1;
            p0 = false;
            qn += __builtin_popcountll(who);
            if (qn >= 64) drain();
        }
    };

    struct Pair { uint4 a, b; };
    // one tile, in buffer h; SEED: instead of the thresholds, what comes closest in this tile passes
    auto scan_tile = [&](auto hc, auto seed_c, int t, bool more) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        constexpr bool SEED = decltype(seed_c)::value;
        uint32_t tw[TW];
#pragma unroll
        for (int i = 0; i < TW; ++i) tw[i] = thr_s[c * TW + i];
        auto issue = [&](int step) -> Pair {
            const int r = step / M, m = step % M;
            const uint32_t ad = row_of(r, m), po = (uint32_t)(m % (M / 2)) * STRIDE + h * FILTER_PLANE;
            Pair p;
            p.a = *reinterpret_cast<const uint4*>(tb + ad + po);
            p.b = *reinterpret_cast<const uint4*>(tb + (ad ^ 32u) + po);
            return p;
        };
        Pair ring[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) ring[d] = issue(d);
        uint32_t acc[2][8], all[2];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (BUFFERS == 2 && !SEED) {
#pragma unroll
                for (int j = 0; j < M * CHUNKS; ++j)
                    if ((j * R) / (2 * M * CHUNKS) == r && more) fetch(t + 1, h ^ 1, j);
            }
            uint32_t (&a)[8] = acc[r & 1];
            uint32_t ts = __builtin_amdgcn_perm(tw[r / 4], tw[r / 4], 0x01010101u * (uint32_t)(r & 3));
            // sums of the bounds, two subspaces per three-operand add; M = 4 adds the code's byte with the last
            auto take = [&](int step) -> Pair {
                const Pair p = ring[step % DEPTH];
                if (step + DEPTH < M * R) ring[step % DEPTH] = issue(step + DEPTH);
                return p;
            };
            {
                const Pair p0 = take(M * r), p1 = take(M * r + 1), p2 = take(M * r + 2);
                a[0] = p0.a.x + p1.a.x + p2.a.x;  a[1] = p0.a.y + p1.a.y + p2.a.y;
                a[2] = p0.a.z + p1.a.z + p2.a.z;  a[3] = p0.a.w + p1.a.w + p2.a.w;
                a[4] = p0.b.x + p1.b.x + p2.b.x;  a[5] = p0.b.y + p1.b.y + p2.b.y;
                a[6] = p0.b.z + p1.b.z + p2.b.z;  a[7] = p0.b.w + p1.b.w + p2.b.w;
            }
#pragma unroll
            for (int m = 3; m + 1 < M; m += 2) {
                const Pair p0 = take(M * r + m), p1 = take(M * r + m + 1);
                a[0] = a[0] + p0.a.x + p1.a.x;  a[1] = a[1] + p0.a.y + p1.a.y;
                a[2] = a[2] + p0.a.z + p1.a.z;  a[3] = a[3] + p0.a.w + p1.a.w;
                a[4] = a[4] + p0.b.x + p1.b.x;  a[5] = a[5] + p0.b.y + p1.b.y;
                a[6] = a[6] + p0.b.z + p1.b.z;  a[7] = a[7] + p0.b.w + p1.b.w;
            }
            {
                const Pair p = take(M * r + M - 1);
                const uint32_t e = M == 4 && !SEED ? ts : 0u;
                a[0] = a[0] + p.a.x + e;  a[1] = a[1] + p.a.y + e;  a[2] = a[2] + p.a.z + e;  a[3] = a[3] + p.a.w + e;
                a[4] = a[4] + p.b.x + e;  a[5] = a[5] + p.b.y + e;  a[6] = a[6] + p.b.z + e;  a[7] = a[7] + p.b.w + e;
            }
            if (SEED) {
                // codes that have no distance yet: the threshold is the smallest sum of this tile
                uint32_t mn = 0xffffffffu;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    mn = pk_min_u16(mn, a[j] & 0x00ff00ffu);
                    mn = pk_min_u16(mn, (a[j] >> 8) & 0x00ff00ffu);
                }
                uint32_t low = (mn & 0xffffu) < (mn >> 16) ? (mn & 0xffffu) : (mn >> 16);
                const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)low, 0xB1, 0xf, 0xf, true);
                low = other < low ? other : low;
                if (ts == 0u) ts = (ALL - low) * 0x01010101u;
                if (M == 4) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) a[j] += ts;
                }
            }
            if (M == 8) {
#pragma unroll
                for (int j = 0; j < 8; ++j) a[j] = __builtin_amdgcn_lerp(a[j], ts, 0x01010101u);
            }
            all[r & 1] = (((a[0] & a[1] & a[2]) & (a[3] & a[4])) & (a[5] & a[6])) & a[7];
            if ((r & 1) && __builtin_expect(__any((all[0] & all[1] & HI) != HI), 0))
                push(acc[0], acc[1], all[0], all[1], r - 1, r, t);
        }
    };

    if (f.seeded == 0 || f.seeded == 3) {
        wait_vector_loads();
        __syncthreads();
        scan_tile(IntC<0>{}, IntC<1>{}, 0, false);
        while (qn > 0) drain();
    }
    int t = 0;
    bool bail = false;
    for (; t < f.ntiles; ++t) {
        wait_vector_loads();
        // one thread says for all whether a wave has run out of its budget; its verdict of this turn stays untouched until
        // everybody has passed the next barrier
        if (tid == 0) bail_s[t & 1] = quit_s;
        __syncthreads();
        if (bail_s[t & 1]) { bail = true; break; }
        const bool more = t + 1 < f.ntiles;
        allowed = filter_budget<M>(t, f.ntiles, later) * (float)C;
        if (BUFFERS == 2 && (t & 1)) scan_tile(IntC<BUFFERS - 1>{}, IntC<0>{}, t, more);
        else scan_tile(IntC<0>{}, IntC<0>{}, t, more);
        if (BUFFERS == 1 && more) {
            __syncthreads();                     // nobody reads this tile any more
#pragma unroll
            for (int j = 0; j < M * CHUNKS; ++j) fetch(t + 1, 0, j);
        }
    }
    if (!bail)
        while (qn > 0) drain();

    // results: lane l finishes the codes l, l + THREADS, ...
    if (BUCKET && tid < 256) gcnt[tid] = 0u;
    wait_vector_loads();
    __syncthreads();
    if (quit_s) {
        give_up();
        return;
    }
#pragma unroll 4
    for (int i = 0; i < R / 2; ++i) {
        const int jj = i * THREADS + tid;
        const int64_t n = base + jj;
        uint32_t pk = 0u, og = ORIGIN_NONE, k = 0u;
        if (n < N) {
            const FilterCode<M> g(gco[n]);
            const unsigned long long key = __hip_atomic_load(&f.state[n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            pk = g.w[0];
            og = g.origin;
            k = key == FILTER_NONE ? 0u : (uint32_t)key;
            if (og != ORIGIN_NONE) {
                assign[og] = (int32_t)k;
                if (dist) {
                    float s = key == FILTER_NONE ? INFINITY : filter_key_distance(key);
                    if (s == 0.0f) s = filter_distance<M>(f.tables, g.w, cen[k]);       // the sign of a zero
                    dist[og] = s;
                }
                if (ro.count) ro.rank[og] = atomicAdd(&ro.count[k], 1u);
            }
        }
        if (BUCKET) {
            // the code, its center, its cluster group and its rank among the workgroup's codes of that group
            uint32_t g = 0xffffffffu, rank = 0u;
            if (og != ORIGIN_NONE) {
                g = k / (uint32_t)bo.KT;
                g = g < 255u ? g : 255u;
                rank = atomicAdd(&gcnt[g], 1u);
            }
            reinterpret_cast<uint4*>(tile)[jj] = make_uint4(pk, k, g, rank);
        }
    }
    if (BUCKET) {
        static_assert(!BUCKET || C * 16 <= TILE_BYTES, "one 16-byte record per code");
        __syncthreads();
        if (tid < 64) {                                          // exclusive prefix over the groups: lane l owns 4l .. 4l+3
            const uint32_t a0 = gcnt[4 * tid], a1 = gcnt[4 * tid + 1], a2 = gcnt[4 * tid + 2], a3 = gcnt[4 * tid + 3];
            const uint32_t mine = a0 + a1 + a2 + a3;
            const uint32_t e0 = wave_inclusive_scan(mine) - mine, e1 = e0 + a0, e2 = e1 + a1, e3 = e2 + a2;
            gbase[4 * tid] = e0;  gbase[4 * tid + 1] = e1;  gbase[4 * tid + 2] = e2;  gbase[4 * tid + 3] = e3;
            const size_t nw = gridDim.x;
            uint2* sg = bo.seg + blockIdx.x;
            if (4 * tid < bo.ngroups) sg[(size_t)(4 * tid) * nw] = make_uint2((uint32_t)(base + e0), a0);
            if (4 * tid + 1 < bo.ngroups) sg[(size_t)(4 * tid + 1) * nw] = make_uint2((uint32_t)(base + e1), a1);
            if (4 * tid + 2 < bo.ngroups) sg[(size_t)(4 * tid + 2) * nw] = make_uint2((uint32_t)(base + e2), a2);
            if (4 * tid + 3 < bo.ngroups) sg[(size_t)(4 * tid + 3) * nw] = make_uint2((uint32_t)(base + e3), a3);
        }
        __syncthreads();
#pragma unroll 2
        for (int i = 0; i < R / 2; ++i) {
            const uint4 r = reinterpret_cast<const uint4*>(tile)[i * THREADS + tid];
            if (r.z != 0xffffffffu) bo.pool[base + gbase[r.z] + r.w] = make_uint2(r.x, r.y);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// M = 16, 32: any order of the codes.  A tile is 64 centers; its subspaces pass through the LDS in phases of four, 64 KB
// each (row (x, s) of 64 bytes at byte x * 256 + s * 64, s = 0..3), two buffers, the next phase's loads straight into LDS
// beside the scan.  Slots of two lanes as in the other scans; of the eight slots an LDS access serves two belong to each
// class j = 0..3, and class j reads subspace (t + j) mod 4 in step t, so that the four classes are in four different bank
// quarters whatever their subcodes are, and of the two slots of a class one starts with the lower half of its rows, the
// other with the upper: no conflicts.  (The order of integer additions is free; the fp32 scans pay three dummy steps per
// tile for the same skew.)  A phase's four subcodes come as one word per code, rotated for the slot's class beforehand, and
// one byte permutation makes an address of a subcode and the lane's constant of the step.  Bounds have 6 bits; the sum of
// a phase's four fits a byte and is added to 16-bit sums in registers, two per instruction, which start at 0x7fff -
// threshold: bit 15 ends up clear exactly when the center passes.
// Candidates as in the scans above.  A code starts from its center of the previous iteration (`assign`), or from the
// closest of the centers that share one of its first FILTER_WIDE_PAIRS pairs of subcodes, or else from the smallest sum
// of the first tile.  A launch covers a round of workgroups and the tiles of 4 MB: all rounds pass over them before
// the next ones, so that they come from the L2 (a phase is scanned in less than the time a load from memory takes, and one
// phase is all there is room to load ahead); keys and the count of candidates carry over from one launch to the next.  A
// workgroup that has used up its budget sets *gave_up, those of later launches stop at once when they see it, and the plain
// scan that is launched behind this one does all the work.
// A phase of 1024 codes is short (0.8 us of work in 1.9 us): either its fill (64 KB per compute unit in that time are 8.8 TB/s out
// of the L2) or its barrier and the start of its reads bound it, and more codes do not fit the registers.
// Measured against the sliding-window scan, M = 32, N = 1e6, K = 1e4: 16.4 -> 12.4 ms in a first iteration, 12.1 and
// 9.5 ms in later ones.
// ---------------------------------------------------------------------------------------------
constexpr int FILTER_WIDE_PAIRS = 3;

// S[phase][position]: the four subcodes of a phase, byte t = subcode (t + j) mod 4 for the position's class j
template <int M>
__global__ __launch_bounds__(256) void code_rotate_kernel(const uint8_t* __restrict__ codes, int64_t N,
                                                          uint32_t* __restrict__ S, int64_t n_alloc,
                                                          const uint32_t* __restrict__ only_if = nullptr)
{
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= n_alloc || (only_if && *only_if == 0u)) return;
    const uint32_t turn = 8u * (uint32_t)((n & 7) >> 1);
    const uint32_t* cw = reinterpret_cast<const uint32_t*>(codes + (n < N ? n : N - 1) * M);
#pragma unroll
    for (int ph = 0; ph < M / 4; ++ph) S[(size_t)ph * n_alloc + n] = __builtin_amdgcn_alignbit(cw[ph], cw[ph], turn);
}

struct FilterWideIn {
    const uint4* img;
    const uint32_t* S;               // rotated subcode words, n_alloc positions per phase
    int64_t n_alloc;
    const uint8_t* codes;            // 4-byte aligned
    const uint8_t* centers;          // 4-byte aligned
    const float* tables;
    const FilterScale* scale;
    unsigned long long* state;
    const uint32_t* pairs;           // [FILTER_WIDE_PAIRS][65536], or NULL
    uint32_t* gave_up;
    uint32_t* spent;                 // per workgroup: candidates formed in the launches before
    int K;
    int t_begin, t_end, ntiles;      // tiles of this launch; the keys hold the result of the tiles before them
    int seeded;                      // assign[] holds a center for every code
    const uint32_t* only_if;         // the scan runs unless this names a word that is 0
};

template <int M>
__device__ __forceinline__ float filter_wide_distance(const float* __restrict__ tables, const uint8_t* __restrict__ x,
                                                      const uint8_t* __restrict__ c)
{
    const uint32_t* xw = reinterpret_cast<const uint32_t*>(x);
    const uint32_t* cw = reinterpret_cast<const uint32_t*>(c);
    float s = 0.0f;
#pragma unroll
    for (int h = 0; h < M; h += 16) {                    // sixteen entries in flight
        float a[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int m = h + i;
            a[i] = tables[((uint32_t)m << 16) | (((xw[m / 4] >> (8 * (m % 4))) & 255u) << 8) | ((cw[m / 4] >> (8 * (m % 4))) & 255u)];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) s = h + i == 0 ? a[0] : s + a[i];
    }
    return s;
}

template <int M, int R, int THREADS>
__global__ __launch_bounds__(THREADS) void assign_filter_wide_kernel(int64_t N, FilterWideIn f, int32_t* __restrict__ assign,
                                                                  float* __restrict__ dist, int64_t first_workgroup)
{
    constexpr int SLOTS = THREADS / 2, C = SLOTS * R, DEPTH = 3, NPH = M / 4;
    constexpr int CHUNKS = 65536 / (THREADS * 16);       // loads per phase
    constexpr uint32_t ALL = M * FILTER_Q_WIDE, DEAD = 0x8000u, HI = 0x80008000u;
    static_assert(NPH % 2 == 0 && R % 2 == 0, "two buffers; every lane finishes R / 2 codes");
    __shared__ float4 tile[TILE_F4];
    __shared__ uint16_t thr_s[SLOTS * R];
    __shared__ uint2 queue_s[THREADS / 64][FILTER_QUEUE];
    __shared__ uint32_t spent_s, quit_s, stop_s[2];
    const char* tb = reinterpret_cast<const char*>(tile);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = tid & 1, c = tid >> 1;
    const uint32_t hq = ((uint32_t)(c & 1) << 5) | ((uint32_t)q << 4);
    const int64_t base = ((int64_t)blockIdx.x + first_workgroup) * C;
    uint2* queue = queue_s[wave];

    const uint64_t ip = reinterpret_cast<uint64_t>(f.img);
    const v4i rs_img = {(int)(uint32_t)ip, (int)(uint32_t)(ip >> 32), (int)((uint32_t)f.ntiles * (uint32_t)NPH * 65536u), 0x00020000};
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)tile;
    const uint32_t wave_off = (uint32_t)wave * 1024u, lane_off = (uint32_t)tid * 16u;
    auto fetch = [&](int gph, int h, int j) {            // part j of phase gph (counted over all tiles) into buffer h
        buffer_to_lds16(lds0 + (uint32_t)h * 65536u + (uint32_t)(j * THREADS * 16) + wave_off, rs_img, lane_off,
                        (uint32_t)gph * 65536u + (uint32_t)(j * THREADS * 16));
    };
#pragma unroll
    for (int j = 0; j < CHUNKS; ++j) fetch(f.t_begin * NPH, 0, j);

    // byte t: the lane's offset inside a 256-byte row group in step t
    uint32_t ub = 0u;
#pragma unroll
    for (int t = 0; t < 4; ++t) ub |= ((((uint32_t)t + ((uint32_t)(c & 7) >> 1)) & 3u) * 64u + hq) << (8 * t);

    const FilterScale sc = *f.scale;
    const int64_t workgroup = (int64_t)blockIdx.x + first_workgroup;
    if (tid == 0) {
        spent_s = f.t_begin > 0 ? f.spent[workgroup] : 0u;
        // one gave up already, or tables that the bounds say nothing about
        quit_s = __hip_atomic_load(f.gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) || !(sc.inv > 0.0f) ? 1u : 0u;
        if (f.only_if && *f.only_if == 0u) quit_s = 2u;      // nothing to do (asked here, beside the other loads: 0.5 us per launch)
    }
    if (tid < 2) stop_s[tid] = 0u;
    __syncthreads();
    if (quit_s) {
        wait_vector_loads();                             // nothing may land in LDS after the workgroup has ended
        if (tid == 0 && quit_s == 1u) *f.gave_up = 1u;
        return;
    }

    // keys and thresholds
#pragma unroll 1
    for (int i = 0; i < R / 2; ++i) {
        const int jj = i * THREADS + tid;
        const int64_t n = base + jj;
        uint32_t bias = DEAD;
        if (n < N) {
            const uint8_t* x = f.codes + n * M;
            float s = INFINITY;
            uint32_t k = 0xffffffffu;
            if (f.t_begin > 0) {
                const unsigned long long key = f.state[n];
                if (key != FILTER_NONE) { s = filter_key_distance(key); k = (uint32_t)key; }
            } else if (f.seeded) {
                k = (uint32_t)assign[n];
                k = k < (uint32_t)f.K ? k : 0u;
                s = filter_wide_distance<M>(f.tables, x, f.centers + (size_t)k * M);
            } else if (f.pairs) {
                uint32_t cand[FILTER_WIDE_PAIRS];
#pragma unroll
                for (int p = 0; p < FILTER_WIDE_PAIRS; ++p)
                    cand[p] = f.pairs[p * 65536 + reinterpret_cast<const uint16_t*>(x)[p]];
#pragma unroll
                for (int p = 0; p < FILTER_WIDE_PAIRS; ++p)
                    if (cand[p] < (uint32_t)f.K && cand[p] != k) {
                        const float d = filter_wide_distance<M>(f.tables, x, f.centers + (size_t)cand[p] * M);
                        if (d < s || (d == s && cand[p] < k)) { s = d; k = cand[p]; }
                    }
            }
            const bool known = s < INFINITY;
            if (f.t_begin == 0) f.state[n] = known ? filter_key(s, k) : FILTER_NONE;
            bias = known ? 0x7fffu - filter_threshold(s, sc, ALL) : 0x7fffu - ALL;
        }
        thr_s[(jj % SLOTS) * R + jj / SLOTS] = (uint16_t)bias;
    }

    int qn = 0;
    // candidates that the workgroup may have formed up to the tile at hand
    float allowed = filter_budget<M>(f.t_begin, f.ntiles, f.seeded != 0) * (float)C;
    auto drain = [&]() __attribute__((always_inline)) {
        if ((float)__builtin_amdgcn_readfirstlane(spent_s) > allowed) {
            quit_s = 1u;
            qn = 0;
            return;
        }
        const int cnt = qn < 64 ? qn : 64;
        qn -= cnt;
        __builtin_amdgcn_wave_barrier();
        const uint2 e = queue[qn + (lane < cnt ? lane : 0)];
        __builtin_amdgcn_wave_barrier();
        uint32_t mask = lane < cnt ? e.x : 0u;
        const uint32_t r = e.y & 31u, sl = (e.y >> 5) & 31u, eq = (e.y >> 10) & 1u, t = e.y >> 11;
        const int slot = wave * 32 + (int)sl;
        const int64_t n = base + (int64_t)r * SLOTS + slot;              // only positions below N ever pass
        const uint32_t piece = 2u * (sl & 1u) + eq;
        const unsigned long long known = __hip_atomic_load(&f.state[n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        {
            const uint32_t in = (uint32_t)known - t * FILTER_TK;
            if (known != FILTER_NONE && in < (uint32_t)FILTER_TK && ((in >> 4) & ~2u) == (piece & ~2u)) {
                const uint32_t j = (((in >> 4) == piece) ? 0u : 4u) + ((in >> 2) & 3u);
                mask &= ~(1u << (8u * (in & 3u) + 7u - j));
            }
        }
        float sb = INFINITY;
        uint32_t kb = 0xffffffffu;
        uint32_t formed = 0u;
#pragma unroll 1
        while (true) {
            const uint64_t who = __ballot(mask != 0u);
            if (!who) break;
            formed += (uint32_t)__builtin_popcountll(who);
            if (mask) {
                const uint32_t bit = (uint32_t)__builtin_ctz(mask), j = 7u - (bit & 7u);
                mask &= mask - 1u;
                const uint32_t k = t * FILTER_TK + 16u * (piece ^ ((j >> 2) << 1)) + 4u * (j & 3u) + (bit >> 3);
                if (k < (uint32_t)f.K) {
                    const float s = filter_wide_distance<M>(f.tables, f.codes + n * M, f.centers + (size_t)k * M);
                    if (s < INFINITY && (s < sb || (s == sb && k < kb))) { sb = s; kb = k; }
                }
            }
        }
        if (kb != 0xffffffffu) {
            atomicMin(&f.state[n], filter_key(sb, kb));
            const uint16_t bias = (uint16_t)(0x7fffu - filter_threshold(sb, sc, ALL));
            uint16_t* p = thr_s + slot * R + r;
            if (bias > *p) *p = bias;
        }
        if (lane == 0) atomicAdd(&spent_s, formed);
    };

    // 16-bit sums of the lane's 32 centers: odd[j] bytes 1 and 3 of word j; all[j] whole words, modulo 2^32, from which the odd bytes'
    // sums leave those of bytes 0 and 2 at the end of a tile: all - (odd << 8).  Five instructions per word and phase instead of seven.
    struct Sums { uint32_t all[8], odd[8]; };
    uint32_t w[R], wn[R];
    auto load_words = [&](int ph) {
#pragma unroll
        for (int r = 0; r < R; ++r) wn[r] = f.S[(size_t)ph * f.n_alloc + base + (int64_t)r * SLOTS + c];
    };
    load_words(0);

    bool stop = false, first = !f.seeded && f.t_begin == 0;   // first: a pass over tile 0 that only finds bounds
    int t = f.t_begin;
    while (t < f.t_end) {
        Sums a[R];
        uint32_t bias[R];
#pragma unroll 1
        for (int ph2 = 0; ph2 < NPH; ph2 += 2) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int ph = ph2 + h;
                wait_vector_loads();
                // one thread decides for all; its verdict of this turn stays until everybody has passed the next barrier
                if (tid == 0) stop_s[h] = quit_s;
                __syncthreads();
                if (stop_s[h]) { stop = true; break; }
#pragma unroll
                for (int r = 0; r < R; ++r) w[r] = wn[r];
                const bool last = ph == NPH - 1;
                const int next = last && first ? 0 : t * NPH + ph + 1;                 // tile 0 again after its first pass
                const bool more = next < f.t_end * NPH;
                load_words(last ? 0 : ph + 1);
                if (ph == 0) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        bias[r] = (uint32_t)thr_s[c * R + r] * 0x10001u;
                        const uint32_t start = first ? 0u : bias[r];
#pragma unroll
                        for (int j = 0; j < 8; ++j) { a[r].all[j] = start + (start << 8); a[r].odd[j] = start; }
                    }
                }
                struct Pair { uint4 a, b; };
                auto issue = [&](int step) -> Pair {
                    const int r = step / 4, tt = step % 4;
                    // (subcode << 8) | the step's offset
                    const uint32_t ad = __builtin_amdgcn_perm(w[r], ub, 0x0c0c0000u | ((uint32_t)(4 + tt) << 8) | (uint32_t)tt) + (uint32_t)h * 65536u;
                    Pair p;
                    p.a = *reinterpret_cast<const uint4*>(tb + ad);
                    p.b = *reinterpret_cast<const uint4*>(tb + (ad ^ 32u));
                    return p;
                };
                Pair ring[DEPTH];
#pragma unroll
                for (int d = 0; d < DEPTH; ++d) ring[d] = issue(d);
#pragma unroll
                for (int r = 0; r < R; ++r) {
#pragma unroll
                    for (int j = 0; j < CHUNKS; ++j)
                        if ((j * R) / (2 * CHUNKS) == r && more) fetch(next, h ^ 1, j);
                    auto take = [&](int step) -> Pair {
                        const Pair p = ring[step % DEPTH];
                        if (step + DEPTH < 4 * R) ring[step % DEPTH] = issue(step + DEPTH);
                        return p;
                    };
                    uint32_t s[8];
                    {
                        const Pair p0 = take(4 * r), p1 = take(4 * r + 1), p2 = take(4 * r + 2);
                        s[0] = p0.a.x + p1.a.x + p2.a.x;  s[1] = p0.a.y + p1.a.y + p2.a.y;
                        s[2] = p0.a.z + p1.a.z + p2.a.z;  s[3] = p0.a.w + p1.a.w + p2.a.w;
                        s[4] = p0.b.x + p1.b.x + p2.b.x;  s[5] = p0.b.y + p1.b.y + p2.b.y;
                        s[6] = p0.b.z + p1.b.z + p2.b.z;  s[7] = p0.b.w + p1.b.w + p2.b.w;
                    }
                    {
                        const Pair p = take(4 * r + 3);
                        s[0] += p.a.x;  s[1] += p.a.y;  s[2] += p.a.z;  s[3] += p.a.w;
                        s[4] += p.b.x;  s[5] += p.b.y;  s[6] += p.b.z;  s[7] += p.b.w;
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        a[r].all[j] += s[j];
                        a[r].odd[j] += __builtin_amdgcn_perm(0u, s[j], 0x0c030c01u);
                    }
                }
            }
            if (stop) break;
        }
        if (stop) break;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t even[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) even[j] = a[r].all[j] - (a[r].odd[j] << 8);
            if (first) {
                // codes without a distance yet: what is closest by the bounds passes; the others' own threshold
                uint32_t mn = 0xffffffffu;
#pragma unroll
                for (int j = 0; j < 8; ++j) mn = pk_min_u16(mn, pk_min_u16(even[j], a[r].odd[j]));
                uint32_t low = (mn & 0xffffu) < (mn >> 16) ? (mn & 0xffffu) : (mn >> 16);
                const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)low, 0xB1, 0xf, 0xf, true);
                low = other < low ? other : low;
                const uint32_t add = (bias[r] & 0xffffu) == 0x7fffu - ALL ? (0x7fffu - low) * 0x10001u : bias[r];
#pragma unroll
                for (int j = 0; j < 8; ++j) { even[j] += add; a[r].odd[j] += add; }
            }
            uint32_t all = HI;
#pragma unroll
            for (int j = 0; j < 8; ++j) all &= even[j] & a[r].odd[j];
            const uint64_t who = __ballot(all != HI);
            if (__builtin_expect(who != 0, 0)) {
                uint32_t m = 0u;                         // bit 8 b + 7 - j: byte b of word j is pruned
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    m |= ((even[j] >> 15) & 0x00010001u) << (7 - j);
                    m |= ((a[r].odd[j] >> 15) & 0x00010001u) << (15 - j);
                }
                m = ~m;
                const int at = qn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
                if (m) queue[at] = make_uint2(m, (uint32_t)r | ((uint32_t)(lane >> 1) << 5) | ((uint32_t)q << 10) | ((uint32_t)t << 11));
                qn += __builtin_popcountll(who);
                if (qn >= 64) drain();
            }
        }
        if (first) {
            while (qn > 0) drain();
            first = false;
        } else {
            ++t;
            if (t < f.ntiles) allowed = filter_budget<M>(t, f.ntiles, f.seeded != 0) * (float)C;
        }
    }
    if (!stop)
        while (qn > 0) drain();
    wait_vector_loads();                                 // nothing may land in LDS after the workgroup has ended
    __syncthreads();
    if (quit_s) {
        if (tid == 0) *f.gave_up = 1u;
        return;
    }
    if (f.t_end < f.ntiles) {
        if (tid == 0) f.spent[workgroup] = spent_s;
        return;
    }
#pragma unroll 1
    for (int i = 0; i < R / 2; ++i) {
        const int64_t n = base + i * THREADS + tid;
        if (n >= N) continue;
        const unsigned long long key = __hip_atomic_load(&f.state[n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t k = key == FILTER_NONE ? 0u : (uint32_t)key;
        assign[n] = (int32_t)k;
        if (dist) {
            float s = key == FILTER_NONE ? INFINITY : filter_key_distance(key);
            if (s == 0.0f) s = filter_wide_distance<M>(f.tables, f.codes + n * M, f.centers + (size_t)k * M);   // the sign of a zero
            dist[n] = s;
        }
    }
}

}  // namespace pqkm
