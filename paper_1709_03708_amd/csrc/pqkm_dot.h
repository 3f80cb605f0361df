// Assignment scan on the matrix cores (Eq. 5 over Eq. 3, exact results).
//
// The scans of pqkm_kernels.h and pqkm_filter.h look M table entries up per code and center, in LDS.  Tables of squared
// distances between codewords (Sec. 2.2) are the squared distances of points in few dimensions, and then Eq. 3 is one inner
// product per code and center, d(x, c) = |u_x|^2 + |u_c|^2 - 2 u_x.u_c, whose cost does not depend on M.
//
// Nothing is assumed about the tables.  A call first looks for such points: per subspace a pivoted Cholesky factorisation
// of the Gram matrix (A[0][i] + A[0][j] - A[i][j]) / 2, at most 256 / M columns, moved to the points' mean.  Every entry of the
// tables is then compared with the points (both in dot_points_kernel): `e0` bounds what an entry sum of Eq. 3 can differ by.
// Tables that no such points describe (more dimensions, not symmetric, infinities, NaN) set `left`, and the scans that are launched
// behind do the work as if this one did not exist; they end at once where it is 0.
//
// The bound.  With u' the points rounded to half precision (times a power of two, all below in those units), d_x = |u_x - u'_x|,
// d_c likewise (the largest of the centers), delta = d_x + d_c, v_c = |u'_c|^2 - 2 u'_x.u'_c from the matrix cores,
// X = |u'_x|^2, e = (1.5 dims + 16) 2^-23 (|u'_x| + max|u'_c|)^2 for the fp32 additions of v, X and |u'_c|^2 (each loses at most
// 2^-23 of a partial sum in the matrix cores, truncation allowed for, and half of that elsewhere):
//   - the center b with the smallest v is at most D = sqrt(v_b + X + e) + delta away from x, so the fp32 distance of Eq. 3 that
//     defines the result is at most D^2 + E, E = e0 + M 2^-23 (D^2 + e0);
//   - a center c with that distance or less is at most sqrt(D^2 + 2 E) away, so v_c <= (sqrt(D^2 + 2 E) + delta)^2 + e - X.
// If only b is within that limit it is the answer, whatever its fp32 distance is.  Otherwise the fp32 distances of those within,
// formed from the caller's tables in the order of Eq. 3, decide by (distance, index): the result is that of the plain scans, bit for
// bit, ties included.  2 to 10 per cent of the codes of clustered data have a second center within the limit.
#pragma once
#include "pqkm_filter.h"

namespace pqkm {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

constexpr int DOT_TILE = 32;                      // centers per matrix instruction
constexpr int DOT_PARTS = 16;                     // blocks per subspace of the check
constexpr uint32_t DOT_CHUNK = 17 * 1024;         // bytes of center fragments loaded together: 16 KB and 1 KB of norms
constexpr int DOT_UNIQUE_MAX_K = 65536;           // centers that repeat another are looked for up to this many
constexpr int DOT_LIST = 2048;                    // (code, center) pairs a workgroup can hold
constexpr int DOT_OVER = 64;                      // codes that need all centers
constexpr float DOT_E0_MAX = 0x1p-11f;            // e0 over the mean distance: beyond, the limit would hold too many centers

struct DotState {
    uint32_t left;                                // not zero: the scans behind do the work
    float e0;                                     // in the tables' units
    float scale;                                  // power of two: units of the rounded points
    uint32_t dc2[2], nc2[2];                      // per parity of the iteration: max |u_c - u'_c|^2, max |u'_c|^2, as bits
    unsigned long long formed[2];                 // likewise: fp32 distances formed
    uint32_t some;                                // not zero: the codes whose assignment is -1 are left (MARKS)
};
struct DotStat { int rank; float spread; };       // per subspace: columns found (more than 256 / M: too many), see DOT_COARSE
struct DotCheck { float e0, sum; };               // per part of a subspace: largest difference, sum of the entries

// 128 or 256 dimensions in all (128 / M or 256 / M per subspace), 0: too many
template <int M>
__device__ __forceinline__ int dot_dims(const DotStat* __restrict__ st)
{
    int most = 0;
    for (int m = 0; m < M; ++m) most = st[m].rank > most ? st[m].rank : most;
    return most <= 128 / M ? 128 : most <= 256 / M ? 256 : 0;
}

// the larger of two, NaN if either is
__device__ __forceinline__ float dot_worse(float a, float b) { return b <= a || a != a ? a : b; }

// the largest of a wave's values, in lane 63
__device__ __forceinline__ uint32_t dot_wave_max(uint32_t v)
{
    auto step = [&](uint32_t o) { v = o > v ? o : v; };
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));          // rows of 16 shifted by 1, 2, 4, 8
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));          // last lane of a row to the next row
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
    return v;
}

// Block (m, part): the points of subspace m, which every block of the subspace finds for itself (a launch and a trip through memory
// less), then rows 16 part .. 16 part + 15 of its table against all 256 of them, the halves of those 16 and what rounding took.
//
// The factorisation is serial in its columns, and a column of all 256 points costs two barriers and a row of the tables, 0.9 us.  So
// one wave first factorises the Gram matrix of 64 of the points, a row of it per lane and the factor in registers: where they
// need too many columns, so do all points, and the block is done; else their pivots serve all points, whose rows then come in one go
// (forward substitution), and only columns that the 64 do not span are found one by one.  No more than most_dims / M columns.
// emb[m][x][256 / M] halves and, behind them, the same with the first half of the columns; lost[m][x] = |u - u'|^2.
// Measured, us, against a factorisation of all 256 points by one block per subspace and a launch for the comparison: M = 8 with 16
// columns 29 -> 17 (and a launch), with 32 42 -> 27; M = 16 15 -> 12; M = 32 11 -> 10.  Whole calls whose tables have more than 256
// dimensions pay 35, 22 and 15 -> 14, 10 and 10 us at M = 8, 16 and 32.
//
// Tables of few values (Hamming distances and the like) are those of points, but so many centers are equally far that the fp32
// distances cost more than the plain scans; they are left (dot_centers_kernel).  Few: in every subspace multiples of the smallest
// positive entry among the 64, and the sum of Eq. 3 spreads by less than DOT_COARSE multiples.
// Hamming distances of 8 bits, whole call, plain scan / without this / with it, us: M = 8 (a sum spreads by 4): 156 / 250 / 177 at N =
// 1e5, K = 1000; 557 / 712 / 582 at 1e6, 1000; M = 16 (5.7): 392 / 567 / 405 at 250007, 999.  M = 32 (8) is tried: 1072 / 337 where
// codes are close to centers, 1091 / 1250 where they are not, at 3e5, 1000.
constexpr int DOT_SAMPLE = 64;
constexpr float DOT_COARSE = 6.0f;

template <int M>
__global__ __launch_bounds__(256) void dot_points_kernel(const float* __restrict__ tables, DotStat* __restrict__ st,
                                                         DotCheck* __restrict__ check, _Float16* __restrict__ emb,
                                                         float* __restrict__ lost, DotState* __restrict__ state, int most_dims)
{
    static_assert(M >= 8, "the columns of a lane are registers");
    constexpr int R = 256 / M, S = DOT_SAMPLE, ROWS = L / DOT_PARTS;
    __shared__ float col[R][L];
    __shared__ float gram_s[S][S];
    __shared__ __attribute__((aligned(16))) float low_s[R][R], row_s[ROWS][R];       // the pivots' rows of the factor; rows to compare
    __shared__ float a0_s[L], d_s[L], inv_s[R], pd_s, red_s[2][4];
    __shared__ int piv_s[R], rank_s;
    __shared__ uint32_t red[3][4];
    const int m = (int)blockIdx.x / DOT_PARTS, part = (int)blockIdx.x % DOT_PARTS;
    const int i = threadIdx.x, lane = i & 63, wave = __builtin_amdgcn_readfirstlane(i >> 6);
    auto sample = [](int t) { return (t & 15) | ((t >> 4) << 6); };    // 64 points: four stretches of 16, a cache line of a row each
    const float* A = tables + (size_t)m * (L * L);
    float sam[S / 4], head[M];
#pragma unroll
    for (int j = 0; j < S / 4; ++j) sam[j] = A[sample(wave * (S / 4) + j) * L + sample(lane)];
#pragma unroll
    for (int q = 0; q < M; ++q) head[q] = tables[(size_t)q * (L * L) + i];
    const float a0 = A[i], diag = A[i * (L + 1)], down = A[i * L];
    float d = a0 - 0.5f * diag, top = 0.0f;
    a0_s[i] = a0;
    d_s[i] = d;
    // distances that could not be any points': not zero on the diagonal, not symmetric in the first row and column
    const bool odd = __builtin_fabsf(diag) + __builtin_fabsf(a0 - down) > 1e-3f * __builtin_fabsf(a0) && i > 0;
    // the largest |u|^2 of the subspace, which says where a column is nothing but rounding, and of all subspaces (negative and NaN
    // count as 0)
#pragma unroll
    for (int q = 0; q < M; ++q) top = head[q] > top ? head[q] : top;
    uint32_t v = dot_wave_max(d > 0.0f ? __builtin_bit_cast(uint32_t, d) : 0u);
    uint32_t vt = dot_wave_max(__builtin_bit_cast(uint32_t, top));
    uint32_t least = 0x7f800000u;                                // smallest positive entry
#pragma unroll
    for (int j = 0; j < S / 4; ++j) {
        const uint32_t b = sam[j] > 0.0f ? __builtin_bit_cast(uint32_t, sam[j]) : 0x7f800000u;
        least = b < least ? b : least;
    }
    least = ~dot_wave_max(~least);
    if (lane == 63) {
        red[0][wave] = v;
        red[1][wave] = vt;
        red[2][wave] = least;
    }
    const bool none = __syncthreads_or(odd);
    v = red[0][0];
    vt = red[1][0];
    least = red[2][0];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
        v = red[0][w] > v ? red[0][w] : v;
        vt = red[1][w] > vt ? red[1][w] : vt;
        least = red[2][w] < least ? red[2][w] : least;
    }
    const float stop = __builtin_bit_cast(float, v) * 0x1p-17f;
    // points are at most 2 sqrt(top) from their mean: a power of two that brings that below 2048, so that what the smallest halves may
    // lose (the 2e-3 in the scan's limit) counts for nothing beside the roundings (0.02 where the bound is 128: a tenth)
    const int ex = (int)(vt >> 23) - 127;
    const float scale = ex > -107 && ex < 109 ? __builtin_bit_cast(float, (uint32_t)(127 + 10 - ((ex + 2) >> 1)) << 23) : 0.0f;
    if (blockIdx.x == 0 && i == 0) {
        state->scale = scale;                                    // 0: nothing to go on with
        state->dc2[0] = state->nc2[0] = 0u;
        state->formed[0] = 0ull;
    }
    if (none || scale == 0.0f) {
        if (part == 0 && i == 0) st[m] = DotStat{R + 1, INFINITY};
        return;
    }
#pragma unroll
    for (int j = 0; j < S / 4; ++j) {
        const int row = wave * (S / 4) + j;
        gram_s[row][lane] = 0.5f * (a0_s[sample(row)] + a0_s[sample(lane)] - sam[j]);
    }
    const float unit = 1.0f / __builtin_bit_cast(float, least);
    float first = 0.0f, second = 0.0f;
    bool fine = least == 0x7f800000u;                            // nothing positive among them: says nothing
#pragma unroll
    for (int j = 0; j < S / 4; ++j) {
        const float x = sam[j] * unit;
        fine = fine || !(__builtin_fabsf(x - __builtin_rintf(x)) < 1e-3f);
        first += x;
        second += x * x;
    }
    if (!__any(fine)) {
#pragma unroll
        for (int off = 32; off; off >>= 1) {
            first += __shfl_xor(first, off);
            second += __shfl_xor(second, off);
        }
        if (lane == 0) { red_s[0][wave] = first; red_s[1][wave] = second; }
    }
    float spread = INFINITY;                                     // variance of the entries, in multiples of the smallest
    if (!__syncthreads_or(fine)) {
        const float mean = (red_s[0][0] + red_s[0][1] + red_s[0][2] + red_s[0][3]) * (1.0f / (S * S));
        spread = (red_s[1][0] + red_s[1][1] + red_s[1][2] + red_s[1][3]) * (1.0f / (S * S)) - mean * mean;
    }
    if (wave == 0) {
        float f[R], ds = d_s[sample(lane)];
        int rank = 0, mine = -1;
#pragma unroll
        for (int k = 0; k < R; ++k) f[k] = 0.0f;
#pragma unroll
        for (int k = 0; k <= R; ++k) {
            const uint32_t w = dot_wave_max(ds > 0.0f ? (__builtin_bit_cast(uint32_t, ds) & ~63u) | (uint32_t)lane : (uint32_t)lane);
            const int p = __builtin_amdgcn_readlane((int)w, 63) & 63;
            const float pd = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ds), p));
            if (!(pd > stop) || !(pd < INFINITY)) break;
            if (k == R || (k == R / 2 && most_dims == 128)) {    // no more columns
                if (pd > 8.0f * stop) rank = R + 1;
                break;
            }
            float g[2] = {0.0f, 0.0f};
            const float whole = gram_s[p][lane];
#pragma unroll
            for (int j = 0; j < k; ++j)
                g[j & 1] = __builtin_fmaf(f[j], __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, f[j]), p)), g[j & 1]);
            const float inv = __builtin_amdgcn_rsqf(pd);
            f[k] = (whole - (g[0] + g[1])) * inv;
            ds = lane == p ? 0.0f : __builtin_fmaf(-f[k], f[k], ds);
            mine = lane == p ? k : mine;
            if (lane == 0) {
                piv_s[k] = sample(p);
                inv_s[k] = inv;
            }
            rank = k + 1;
        }
        if (mine >= 0)
#pragma unroll
            for (int k = 0; k < R; ++k) low_s[mine][k] = f[k];
        if (lane == 0) rank_s = rank;
    }
    __syncthreads();
    int rank = __builtin_amdgcn_readfirstlane(rank_s);
    if (rank > R) {
        if (part == 0 && i == 0) st[m] = DotStat{R + 1, INFINITY};
        return;
    }
    float u[R];
#pragma unroll
    for (int k = 0; k < R; ++k) u[k] = k < rank ? A[piv_s[k] * L + i] : 0.0f;
#pragma unroll
    for (int k = 0; k < R; ++k)
        if (k < rank) {
            float g[2] = {0.0f, 0.0f};
#pragma unroll
            for (int j = 0; j < k; ++j) g[j & 1] = __builtin_fmaf(u[j], low_s[k][j], g[j & 1]);
            const int x = piv_s[k];
            u[k] = (0.5f * (a0 + a0_s[x] - u[k]) - (g[0] + g[1])) * inv_s[k];
            col[k][i] = u[k];
            d = i == x ? 0.0f : __builtin_fmaf(-u[k], u[k], d);
        }
    __syncthreads();
    const int columns = most_dims / M;
#pragma unroll 1
    for (int k = rank; k <= columns; ++k) {
        // the largest of what is left, with its row in the low bits; negative and NaN count as 0
        uint32_t w = d > 0.0f ? (__builtin_bit_cast(uint32_t, d) & ~255u) | (uint32_t)i : (uint32_t)i;
        w = dot_wave_max(w);
        if (lane == 63) red[0][wave] = w;
        __syncthreads();
        w = red[0][0];
#pragma unroll
        for (int q = 1; q < 4; ++q) w = red[0][q] > w ? red[0][q] : w;
        const int p = (int)(w & 255u);
        if (i == p) pd_s = d;
        __syncthreads();
        const float pd = pd_s;
        if (!(pd > stop) || !(pd < INFINITY)) break;
        if (k == columns) {
            if (pd > 8.0f * stop) rank = R + 1;
            break;
        }
        const float ap = A[p * L + i];
        float g = 0.0f;
#pragma unroll 8
        for (int j = 0; j < k; ++j) g = __builtin_fmaf(col[j][i], col[j][p], g);
        g = (0.5f * (a0 + a0_s[p] - ap) - g) / __builtin_sqrtf(pd);
        col[k][i] = g;                                           // column k of row p is read behind the next two barriers
        d = i == p ? 0.0f : __builtin_fmaf(-g, g, d);
        rank = k + 1;
    }
    if (part == 0 && i == 0) st[m] = DotStat{rank, spread};
    if (rank > R) return;
    float a[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) a[r] = A[(part * ROWS + r) * L + i];
    __syncthreads();
    // moved to the mean of the 256 points: shorter vectors, smaller roundings
    for (int k = wave; k < rank; k += 4) {
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) s += col[k][lane + 64 * q];
#pragma unroll
        for (int off = 32; off; off >>= 1) s += __shfl_xor(s, off);
        s *= 1.0f / 256.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) col[k][lane + 64 * q] -= s;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R; ++k) u[k] = k < rank ? col[k][i] : 0.0f;
    for (int t = i; t < ROWS * R; t += 256) row_s[t / R][t % R] = t % R < rank ? col[t % R][part * ROWS + t / R] : 0.0f;
    __syncthreads();
    float e0 = 0.0f, sum = 0.0f;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        float q = 0.0f;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const float t = u[k] - row_s[r][k];
            q = __builtin_fmaf(t, t, q);
        }
        // the roundings of q itself: R + 2 of them, each at most 2^-24 of it
        e0 = dot_worse(e0, __builtin_fabsf(a[r] - q) + q * ((float)(R + 8) * 0x1p-23f));
        sum += a[r];
    }
#pragma unroll
    for (int off = 32; off; off >>= 1) {
        e0 = dot_worse(e0, __shfl_xor(e0, off));
        sum += __shfl_xor(sum, off);
    }
    if (lane == 0) { red_s[0][wave] = e0; red_s[1][wave] = sum; }
    // the halves: R = 8, 16 or 32 neighbouring lanes to a row
    for (int at = i; at < ROWS * R; at += 256) {                 // ROWS R is a multiple of 64: whole waves
        const int r = at / R, k = at % R;
        const size_t x = (size_t)m * L + part * ROWS + r;
        const float w = row_s[r][k] * scale;
        const _Float16 h = (_Float16)w;
        float took = (w - (float)h) * (w - (float)h);
#pragma unroll
        for (int off = 1; off < R; off <<= 1) took += __shfl_xor(took, off);
        emb[x * R + k] = h;
        if (k < R / 2) emb[(size_t)L * 256 + x * (R / 2) + k] = h;
        if (k == 0) lost[x] = took * (1.0f + 0x1p-16f);
    }
    __syncthreads();
    if (i == 0) {
        for (int w = 1; w < 4; ++w) {
            e0 = dot_worse(e0, red_s[0][w]);
            sum += red_s[1][w];
        }
        check[blockIdx.x] = DotCheck{e0, sum};
    }
}

// Fragments of a tile of 32 centers, in the order the matrix instruction reads them: chunks of 16 KB (2 tiles of 128
// dimensions or 1 of 256) and 1 KB of norms.  [tile][step of 16 dimensions][lane], -2 u' of center lane % 32, dimensions 8 (lane / 32)
// .. + 7 of the step.  Norms |u'|^2 as the accumulators want them, [tile][lane / 32][register]; +inf past K, and for a center
// that repeats one of a lower index, which it can never be selected over.
// The first launch of a call decides whether the tables are what this scan needs.
template <int M>
__global__ __launch_bounds__(256) void dot_centers_kernel(const uint8_t* __restrict__ centers, int K,
                                                          const DotStat* __restrict__ st, const DotCheck* __restrict__ check,
                                                          const _Float16* __restrict__ emb, const float* __restrict__ lost,
                                                          DotState* __restrict__ state, char* __restrict__ img, int iteration,
                                                          bool decide)
{
    __shared__ float sq_s[32][DOT_TILE], lost_s[8][DOT_TILE];
    __shared__ float e0_s[M], sum_s[M];
    __shared__ uint32_t word_s[DOT_TILE], dup_s[DOT_TILE];
    const int tile = (int)blockIdx.x, t = threadIdx.x;
    const int dims = dot_dims<M>(st);
    const bool usable = dims > 0 && state->scale > 0.0f;
    if (decide) {
        if (blockIdx.x == 0) {
            if (t < M && usable) {
                float e0 = 0.0f, sum = 0.0f;
#pragma unroll
                for (int p = 0; p < DOT_PARTS; ++p) {
                    const DotCheck c = check[t * DOT_PARTS + p];
                    e0 = dot_worse(e0, c.e0);
                    sum += c.sum;
                }
                e0_s[t] = e0;
                sum_s[t] = sum;
            }
            __syncthreads();
            if (t == 0) {
                float e0 = 0.0f, sum = 0.0f, spread = 0.0f;
                if (usable)
                    for (int m = 0; m < M; ++m) { e0 += e0_s[m]; sum += sum_s[m]; spread += st[m].spread; }
                // an infinite entry makes e0 and perhaps the sum infinite, a NaN both NaN
                state->left = usable && e0 < INFINITY && sum < INFINITY && e0 <= DOT_E0_MAX * (sum * (1.0f / 65536.0f)) &&
                              !(spread < DOT_COARSE * DOT_COARSE) ? 0u : 1u;
                state->e0 = e0;
            }
        }
        if (!usable) return;
    } else if (state->left) {
        return;
    }
    if (blockIdx.x == 0 && t == 0) {
        state->dc2[(iteration & 1) ^ 1] = state->nc2[(iteration & 1) ^ 1] = 0u;
        state->formed[(iteration & 1) ^ 1] = 0ull;
        state->some = 0u;
    }
    // which centers repeat one of a lower index, by their first four subcodes and then the rest
    if (t < DOT_TILE) {
        const int64_t k = (int64_t)tile * DOT_TILE + t;
        word_s[t] = k < K ? reinterpret_cast<const uint32_t*>(centers)[k * (M / 4)] : 0u;
        dup_s[t] = 0u;
    }
    __syncthreads();
    if (K <= DOT_UNIQUE_MAX_K) {
        uint32_t w[DOT_TILE];
#pragma unroll
        for (int i = 0; i < DOT_TILE; ++i) w[i] = word_s[i];
        const int last = (tile + 1) * DOT_TILE < K ? (tile + 1) * DOT_TILE : K;
#pragma unroll 4
        for (int j = t; j < last; j += 256) {
            const uint32_t v = reinterpret_cast<const uint32_t*>(centers)[(size_t)j * (M / 4)];
            uint32_t hit = 0u;
#pragma unroll
            for (int i = 0; i < DOT_TILE; ++i) hit |= v == w[i] ? 1u << i : 0u;
            while (hit) {
                const int i = __builtin_ctz(hit), k = tile * DOT_TILE + i;
                hit &= hit - 1u;
                bool same = j < k && k < K;
                for (int q = 1; same && q < M / 4; ++q)
                    same = reinterpret_cast<const uint32_t*>(centers)[(size_t)j * (M / 4) + q] ==
                           reinterpret_cast<const uint32_t*>(centers)[(size_t)k * (M / 4) + q];
                if (same) dup_s[i] = 1u;
            }
        }
    }
    const int r = dims / M, steps = dims / 16;
    if (dims == 128) emb += (size_t)L * 256;                     // the halves of the first columns only
    const int per = 256 / dims;                                  // tiles per chunk
    char* chunk = img + (size_t)(tile / per) * DOT_CHUNK;
    for (int f = t; f < steps * 64; f += 256) {
        const int fl = f & 63, ks = f >> 6;
        const int row = fl & 31, d0 = ks * 16 + 8 * (fl >> 5);
        const int64_t k = (int64_t)tile * DOT_TILE + row;
        v8h v;
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = (_Float16)0.0f;
        if (k < K) {
            if (r >= 8) {
                const int m = d0 / r;
                v = *reinterpret_cast<const v8h*>(emb + ((size_t)m * L + centers[k * M + m]) * r + d0 % r);
            } else {                                             // r = 4
                const int m = d0 / 4;
                const v4h a = *reinterpret_cast<const v4h*>(emb + ((size_t)m * L + centers[k * M + m]) * 4);
                const v4h b = *reinterpret_cast<const v4h*>(emb + ((size_t)(m + 1) * L + centers[k * M + m + 1]) * 4);
                v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
        float sq = 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            sq = __builtin_fmaf((float)v[q], (float)v[q], sq);
            v[q] = (_Float16)-2.0f * v[q];
        }
        sq_s[2 * ks + (fl >> 5)][row] = sq;
        *reinterpret_cast<v8h*>(chunk + ((size_t)(tile % per) * steps * 64 + f) * 16) = v;
    }
    {
        const int row = t & 31, part = t >> 5;
        const int64_t k = (int64_t)tile * DOT_TILE + row;
        float s = 0.0f;
        if (k < K)
            for (int m = part; m < M; m += 8) s += lost[m * L + centers[k * M + m]];
        lost_s[part][row] = s;
    }
    __syncthreads();
    if (t < DOT_TILE) {
        const int64_t k = (int64_t)tile * DOT_TILE + t;
        float n = 0.0f, s = 0.0f;
        for (int q = 0; q < 2 * steps; ++q) n += sq_s[q][t];
        for (int q = 0; q < 8; ++q) s += lost_s[q][t];
        float most_n = k < K ? n : 0.0f, most_s = s;
#pragma unroll
        for (int off = 16; off; off >>= 1) {
            most_n = __builtin_fmaxf(most_n, __shfl_xor(most_n, off));
            most_s = __builtin_fmaxf(most_s, __shfl_xor(most_s, off));
        }
        if (t == 0) {
            atomicMax(&state->nc2[iteration & 1], __builtin_bit_cast(uint32_t, most_n));
            atomicMax(&state->dc2[iteration & 1], __builtin_bit_cast(uint32_t, most_s));
        }
        // row t is register 4 (t / 8) + t % 4 of half t / 4 % 2
        const int half = (t >> 2) & 1, reg = 4 * (t >> 3) + (t & 3);
        reinterpret_cast<float*>(chunk + 16384)[(tile % per) * 32 + half * 16 + reg] = k < K && !dup_s[t] ? n : INFINITY;
    }
    // the chunk's second tile, where there is none
    if (per == 2 && blockIdx.x == gridDim.x - 1 && tile % 2 == 0) {
        for (int f = t; f < 512; f += 256) reinterpret_cast<float4*>(chunk)[512 + f] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (t < 32) reinterpret_cast<float*>(chunk + 16384)[32 + t] = INFINITY;
    }
}

struct DotIn {
    const uint8_t* codes;                         // 4-byte aligned, as the centers
    const uint8_t* centers;
    const float* tables;
    const DotStat* st;
    const _Float16* emb;
    const float* lost;
    const char* img;
    DotState* state;
    int64_t N;
    int K, iteration;
};

// the fp32 distance of Eq. 3
template <int M>
__device__ __forceinline__ float dot_distance(const float* __restrict__ tables, const uint8_t* __restrict__ x,
                                              const uint8_t* __restrict__ c)
{
    const uint32_t* xw = reinterpret_cast<const uint32_t*>(x);
    const uint32_t* cw = reinterpret_cast<const uint32_t*>(c);
    constexpr int W = M < 16 ? M : 16;            // entries in flight
    float s = 0.0f;
#pragma unroll
    for (int h = 0; h < M; h += W) {
        float a[W];
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const int m = h + i;
            a[i] = tables[((uint32_t)m << 16) | (((xw[m / 4] >> (8 * (m % 4))) & 255u) << 8) | ((cw[m / 4] >> (8 * (m % 4))) & 255u)];
        }
#pragma unroll
        for (int i = 0; i < W; ++i) s = h + i == 0 ? a[0] : s + a[i];
    }
    return s;
}

// ---------------------------------------------------------------------------------------------
// The scan.  512 threads, one workgroup per compute unit, which stays for all its codes: the halves of the points are 64 KB
// of LDS (128 dimensions; with 256 the two halves of the subspaces take turns).  A wave takes 32 CT codes as columns, whose
// fragments it gathers from there into 64 registers, and the workgroup passes over the centers (rows) in chunks of 16 KB,
// loaded straight into LDS one chunk ahead.  Per tile of 32 centers and column a lane holds 16 centers of one code: it takes
// their minimum, keeps the four smallest such minima with the tiles of three, and the 16 values under the smallest.  At the end
// the two lanes of a code know the limit, and all but a few codes have one center within.
// The others list the centers of their block within it and all 16 of a second and a third one, and the workgroup works off the
// list together; where there is a fourth block it forms all K.  A workgroup whose codes need so many that the plain scans are cheaper (ties
// everywhere) sets `left` and ends, and so do the others when they next look.  Where the scan behind can take single codes (one lane
// per center) it marks its block's instead and goes on, until half of all codes are marked: with few codes a workgroup has one
// block, and knows at its end.  M = 16, 256 dimensions, N = 33000, K = 6000, one such block of 129: 525 us by the scan behind alone, 800 with all
// codes left to it, 310 with the block's, 285 where there is none.
//
// Per tile and 32 codes 8 matrix instructions (128 dimensions) of 32 clocks and about 40 vector instructions of 4.  Two waves per
// SIMD, whose two kinds of instruction overlap little: at M = 8, N = 5e5, K = 5000 the matrix cores are busy 46 per cent of the
// time and the vector units 28, at 2.0 GHz (the clock falls from 2.4 under this load); LDS reads 18.  Two columns per wave, so that
// a fragment read from LDS serves two instructions; reads run four steps ahead (two in flight: 1.2 times the time).  With few centers
// a block's own cost shows: codes, gather and two barriers with the distances between, 10 to 13 us per 512 codes, so the next block's
// codes are loaded ahead.
// Measured, plain or lower-bound scan -> this with all its launches, us, with distances: M = 16, N = 250007, K = 999: 355 -> 118;
// M = 8, N = 1e6, K = 1000: 574 -> 342; M = 16, N = 4e5, K = 5000: 1752 -> 680; M = 32, N = 3e5, K = 6000: 6850 -> 719.  The kernel
// itself at M = 8, N = 5e5, K = 5000, without distances: 670 to 730 us, 3.4 to 3.7e12 pairs per second.
// ---------------------------------------------------------------------------------------------
template <int M, int DIMS, int CT, bool MARKS>
__device__ __forceinline__ void dot_scan(const DotIn& f, int32_t* __restrict__ assign, float* __restrict__ dist, float4* tab,
                                         float* lost_s, char* buf, unsigned long long* key_s, uint32_t* list_s,
                                         uint32_t* over_s, uint32_t* code_s, uint32_t* misc)
{
    constexpr int KS = DIMS / 16, HALVES = DIMS / 128, PER = 256 / DIMS, R = DIMS / M;
    constexpr int WAVES = 8, C = WAVES * 32 * CT;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = (f.K + DOT_TILE - 1) / DOT_TILE, nchunks = (ntiles + PER - 1) / PER;
    const int64_t nblocks = (f.N + C - 1) / C;

    auto rsrc_of = [&](const void* p, uint32_t bytes) {
        const uint64_t a = reinterpret_cast<uint64_t>(p);
        return v4i{(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)bytes, 0x00020000};
    };
    const v4i rs_img = rsrc_of(f.img, (uint32_t)nchunks * DOT_CHUNK);
    const v4i rs_emb = rsrc_of(f.emb + (DIMS == 128 ? L * 256 : 0), (uint32_t)HALVES * 65536u);
    auto lds_of = [&](const void* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p; };
    const uint32_t buf0 = lds_of(buf), tab0 = lds_of(tab), lane16 = (uint32_t)lane * 16u;
    auto fetch = [&](int chunk, int b) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t at = (uint32_t)(wave + 8 * j) * 1024u;
            buffer_to_lds16(buf0 + (uint32_t)b * DOT_CHUNK + at, rs_img, lane16, (uint32_t)chunk * DOT_CHUNK + at);
        }
        if (wave == (chunk & 7)) buffer_to_lds16(buf0 + (uint32_t)b * DOT_CHUNK + 16384u, rs_img, lane16, (uint32_t)chunk * DOT_CHUNK + 16384u);
    };
    auto fetch_points = [&](int h) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t at = (uint32_t)(wave + 8 * j) * 1024u;
            buffer_to_lds16(tab0 + at, rs_emb, lane16, (uint32_t)h * 65536u + at);
        }
    };
    if (HALVES == 1) fetch_points(0);
    for (int i = tid; i < M * L; i += 512) lost_s[i] = f.lost[i];

    const float scale = f.state->scale, s2 = scale * scale;
    const float e0 = f.state->e0 * s2 * 1.0001f;
    const float dc = __builtin_sqrtf(__builtin_bit_cast(float, f.state->dc2[f.iteration & 1])) * 1.0001f;
    const float nc = __builtin_sqrtf(__builtin_bit_cast(float, f.state->nc2[f.iteration & 1])) * 1.0001f;
    // fp32 distances that may be formed per code: what the plain scan costs, at 5 clocks per entry
    const float free_evals = 0.7f * FilterCost<M>::plain * (float)f.K * (1.0f / 64.0f) / (5.0f * (float)M) + (dist ? 1.0f : 0.0f);
    const float most = 2.0f * free_evals * (float)C + 1024.0f;   // in one block
    float spent = 0.0f, done_codes = 0.0f;
    int gb = 0;                                                  // buffer of the next chunk
    // the codes of a block, one block ahead: C M bytes in pieces of 1 KB, zeros past the end
    const uint32_t code0 = lds_of(code_s);
    auto fetch_codes = [&](int64_t blk) {
        const int64_t left_bytes = (f.N - blk * C) * M;
        const v4i rs = rsrc_of(f.codes + blk * C * M, left_bytes < C * M ? (uint32_t)left_bytes : (uint32_t)(C * M));
        for (int j = wave; j < C * M / 1024; j += WAVES)
            buffer_to_lds16(code0 + (uint32_t)j * 1024u, rs, lane16, (uint32_t)j * 1024u);
    };
    fetch_codes(blockIdx.x);
    fetch(0, 0);

    // seen by the workgroups of other XCDs while this kernel runs, not only behind its end
    auto leave = [&]() { __hip_atomic_store(&f.state->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };

    for (int64_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        const int64_t base = blk * C + wave * (32 * CT);
        // has another workgroup given up?  One thread asks for all
        uint32_t given_up = 0u;
        if (tid == 0) given_up = __hip_atomic_load(&f.state->left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // fragments of the codes
        v8h x[CT][KS];
        float X[CT], lx[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) { X[ct] = 0.0f; lx[ct] = 0.0f; }
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
            if (HALVES == 2) {
                __syncthreads();                                 // the last half is read no more
                fetch_points(h);
            }
            wait_vector_loads();
            __syncthreads();
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const uint32_t* cw = code_s + (wave * (32 * CT) + ct * 32 + col) * (M / 4);
                uint32_t w[M / 4];
#pragma unroll
                for (int i = 0; i < M / 4; ++i) w[i] = cw[i];
                auto sub = [&](int m) -> uint32_t { return (w[m / 4] >> (8 * (m % 4))) & 255u; };
#pragma unroll
                for (int k8 = 0; k8 < 8; ++k8) {
                    const int ks = 8 * h + k8;
                    v8h& v = x[ct][ks];
                    const char* tb = reinterpret_cast<const char*>(tab);
                    if (R >= 16) {
                        const int m = ks * 16 / R, ml = m - h * (M / HALVES);
                        v = *reinterpret_cast<const v8h*>(tb + ((uint32_t)(ml * L) + sub(m)) * (R * 2) + (ks * 16 % R) * 2 + half * 16);
                    } else if (R == 8) {
                        const int m = 2 * ks, ml = m - h * (M / HALVES);
                        const uint32_t s = half ? sub(m + 1) + L : sub(m);
                        v = *reinterpret_cast<const v8h*>(tb + ((uint32_t)(ml * L) + s) * 16);
                    } else {
                        const int m = 4 * ks, ml = m - h * (M / HALVES);
                        const uint32_t sa = half ? sub(m + 2) + 2 * L : sub(m), sb = half ? sub(m + 3) + 2 * L : sub(m + 1);
                        const v4h a = *reinterpret_cast<const v4h*>(tb + ((uint32_t)(ml * L) + sa) * 8);
                        const v4h b = *reinterpret_cast<const v4h*>(tb + ((uint32_t)((ml + 1) * L) + sb) * 8);
                        v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
                    }
#pragma unroll
                    for (int q = 0; q < 8; q += 2) {
                        const v2h p = {v[q], v[q + 1]};
                        X[ct] = __builtin_amdgcn_fdot2(p, p, X[ct], false);
                    }
                }
                // half of the subspaces per lane
                if (h == 0)
#pragma unroll
                    for (int m = 0; m < M / 2; ++m) {
                        const uint32_t s = half ? sub(m + M / 2) : sub(m);
                        lx[ct] += lost_s[(m + half * (M / 2)) * L + (int)s];
                    }
            }
        }
        float b1[CT], b2[CT], b3[CT], b4[CT], kept[CT][16];
        int i1[CT], i2[CT], i3[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            X[ct] += __shfl_xor(X[ct], 32);
            lx[ct] += __shfl_xor(lx[ct], 32);
            b1[ct] = b2[ct] = b3[ct] = b4[ct] = INFINITY;
            i1[ct] = i2[ct] = i3[ct] = 0;
#pragma unroll
            for (int j = 0; j < 16; ++j) kept[ct][j] = INFINITY;
        }
        const bool again = blk + gridDim.x < nblocks;
        __syncthreads();                                         // everybody has its codes
        if (again) fetch_codes(blk + gridDim.x);
#pragma unroll 1
        for (int ch = 0; ch < nchunks; ++ch) {
            wait_vector_loads();
            __syncthreads();
            const int cur = gb;
            gb ^= 1;
            if (ch + 1 < nchunks) fetch(ch + 1, gb);
            else if (again) fetch(0, gb);
            const char* cb = buf + cur * DOT_CHUNK;
            // fragments and norms are read AHEAD steps ahead, over the end of a tile within the chunk
            constexpr int AHEAD = 4;
            auto fragment = [&](int step) { return *reinterpret_cast<const v8h*>(cb + step * 1024 + lane * 16); };
            auto norms = [&](int p) {
                v16f n;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float4 q = *reinterpret_cast<const float4*>(cb + 16384 + p * 128 + half * 64 + j * 16);
                    n[4 * j] = q.x; n[4 * j + 1] = q.y; n[4 * j + 2] = q.z; n[4 * j + 3] = q.w;
                }
                return n;
            };
            v16f cn = norms(0);
            v8h ring[AHEAD];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) ring[i] = fragment(i);
            __builtin_amdgcn_sched_group_barrier(0x100, 4 + AHEAD, 0);
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                const int t = ch * PER + p;
                v16f acc[CT];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const int step = p * KS + ks;
                    const v8h a = ring[step % AHEAD];
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        acc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, x[ct][ks], ks == 0 ? cn : acc[ct], 0, 0, 0);
                    if (step + AHEAD < PER * KS) ring[step % AHEAD] = fragment(step + AHEAD);
                    __builtin_amdgcn_sched_group_barrier(0x008, CT, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                if (p + 1 < PER) cn = norms(p + 1);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const v16f& v = acc[ct];
                    const float u0 = minimum3(v[0], v[1], v[2]), u1 = minimum3(v[3], v[4], v[5]);
                    const float u2 = minimum3(v[6], v[7], v[8]), u3 = minimum3(v[9], v[10], v[11]);
                    const float u4 = minimum3(v[12], v[13], v[14]);
                    const float e = minimum3(minimum3(u0, u1, u2), minimum3(u3, u4, v[15]), u0);
                    const bool f1 = e < b1[ct], f2 = e < b2[ct], f3 = e < b3[ct];
                    b4[ct] = __builtin_amdgcn_fmed3f(b3[ct], b4[ct], e);
                    b3[ct] = __builtin_amdgcn_fmed3f(b2[ct], b3[ct], e);
                    b2[ct] = __builtin_amdgcn_fmed3f(b1[ct], b2[ct], e);
                    b1[ct] = f1 ? e : b1[ct];
                    const int n3 = __builtin_unpredictable(f3) ? t : i3[ct], n2 = __builtin_unpredictable(f2) ? t : i2[ct];
                    i3[ct] = __builtin_unpredictable(f2) ? i2[ct] : n3;
                    i2[ct] = __builtin_unpredictable(f1) ? i1[ct] : n2;
                    i1[ct] = f1 ? t : i1[ct];
#pragma unroll
                    for (int j = 0; j < 16; ++j) kept[ct][j] = f1 ? v[j] : kept[ct][j];
                }
            }
        }

        // the centers within the limit: one, which is the answer, or several, which are listed for the whole workgroup
        unsigned long long* keys = key_s + wave * (32 * CT);
        if (lane < 32 * CT) keys[lane] = FILTER_NONE;
        __builtin_amdgcn_wave_barrier();
        auto center_of = [&](int t, int h, int j) { return (uint32_t)(t * DOT_TILE + 8 * (j >> 2) + 4 * h + (j & 3)); };
        auto form = [&](int c, uint32_t k) __attribute__((always_inline)) {
            const float s = dot_distance<M>(f.tables, f.codes + (blk * C + c) * M, f.centers + (size_t)k * M);
            if (s < INFINITY) atomicMin(&key_s[c], filter_key(s, k));
        };
        auto append = [&](bool mine, int c, uint32_t k) __attribute__((always_inline)) {
            mine = mine && k < (uint32_t)f.K;
            const uint64_t who = __ballot(mine);
            if (!who) return;
            uint32_t at = 0u;
            if (lane == 0) at = atomicAdd(&misc[2], (uint32_t)__builtin_popcountll(who));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
                 __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
            if (!mine) return;
            if (at < (uint32_t)DOT_LIST) list_s[at] = (uint32_t)c | (k << 9);
            else if ((float)at < most) form(c, k);               // no room; from `most` on the codes are left anyway
        };
        const int c0 = wave * (32 * CT);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const int64_t n = base + ct * 32 + col;
            const bool live = n < f.N;
            const float best = min_f32(b1[ct], __shfl_xor(b1[ct], 32));
            const float rx = __builtin_sqrtf(X[ct]) * 1.0001f + nc;
            const float e = (1.5f * (float)DIMS + 16.0f) * 0x1p-23f * rx * rx + 1e-30f;
            const float delta = __builtin_sqrtf(lx[ct]) * 1.0001f + dc + 2e-3f;          // denormal halves may count as 0
            const float D = __builtin_sqrtf(__builtin_fmaxf(best + X[ct], 0.0f) + e) * 1.00001f + delta;
            const float E = e0 + (float)M * 0x1p-23f * (D * D + e0);
            const float far = __builtin_sqrtf(D * D * 1.00001f + 2.0f * E) * 1.00001f + delta;
            const float lim = far * far * 1.00001f + e - X[ct];
            uint32_t mask = 0u;
#pragma unroll
            for (int j = 0; j < 16; ++j) mask |= kept[ct][j] <= lim ? 1u << j : 0u;
            const bool two = b2[ct] <= lim, three = b3[ct] <= lim;
            bool over = b4[ct] <= lim;
            int total = __builtin_popcount(mask) + (two ? 16 : 0);
            total += __shfl_xor(total, 32);
            over = __shfl_xor((int)over, 32) || over || total == 0;
            if (!live) { mask = 0u; over = false; }
            if (total == 1 && !over && !dist) {
                if (mask) keys[ct * 32 + col] = center_of(i1[ct], half, __builtin_ctz(mask));
                mask = 0u;
            }
            if (over) mask = 0u;
            while (__any(mask != 0u)) {
                append(mask != 0u, c0 + ct * 32 + col, center_of(i1[ct], half, __builtin_ctz(mask | 0x10000u)));
                mask &= mask - 1u;
            }
            // second and third blocks: four at a time, 16 lanes each
            auto block = [&](uint64_t who, int tile_of) __attribute__((always_inline)) {
                while (who) {
                    int src = -1;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int b = who ? __builtin_ctzll(who) : -1;
                        who &= who - 1;
                        if (lane >> 4 == q) src = b;
                    }
                    const int t = __shfl(tile_of, src < 0 ? 0 : src);
                    append(src >= 0, c0 + ct * 32 + (src & 31), center_of(t, (src >> 5) & 1, lane & 15));
                }
            };
            block(__ballot(two && live && !over), i2[ct]);
            block(__ballot(three && live && !over), i3[ct]);
            if (over && half == 0) {
                const uint32_t at = atomicAdd(&misc[3], 1u);
                if (at < (uint32_t)DOT_OVER) over_s[at] = (uint32_t)(c0 + ct * 32 + col);
            }
        }
        __syncthreads();
        const uint32_t listed = misc[2], overs = misc[3];
        // far more than the plain scan of these codes would cost: the same verdict in all threads
        const float cost = (float)listed + (float)overs * (float)f.K;
        const bool over = overs > (uint32_t)DOT_OVER || cost > most, beyond = MARKS && over;
        if (over && !MARKS) {
            if (tid == 0) leave();
            break;
        }
        if (beyond) {
            if (tid == 0) __hip_atomic_store(&f.state->some, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            for (uint32_t i = (uint32_t)tid; i < (listed < (uint32_t)DOT_LIST ? listed : (uint32_t)DOT_LIST); i += 512u) {
                const uint32_t e = list_s[i];
                form((int)(e & 511u), e >> 9);
            }
            for (uint32_t i = 0; i < overs; ++i) {
                const int c = (int)over_s[i];
#pragma unroll 4
                for (int k = tid; k < f.K; k += 512) form(c, (uint32_t)k);
            }
        }
        // more than this workgroup's share of what the plain scan would cost: told to the others, and half of the whole is enough
        spent += beyond ? 1.01f * free_evals * (float)C : cost;
        done_codes += (float)C;
        if (spent > free_evals * done_codes) {
            if (tid == 0) {
                const unsigned long long all = atomicAdd(&f.state->formed[f.iteration & 1], (unsigned long long)spent);
                if ((float)all + spent > 0.5f * free_evals * (float)f.N) {
                    leave();
                    given_up = 1u;
                }
            }
            spent = done_codes = 0.0f;
        }
        if (tid == 0) misc[1] = again ? given_up : 0u;
        __syncthreads();
        if (lane < 32 * CT) {
            const int64_t n = base + lane;
            if (n < f.N) {
                const unsigned long long key = keys[lane];
                const uint32_t k = key == FILTER_NONE ? 0u : (uint32_t)key;
                assign[n] = beyond ? -1 : (int32_t)k;
                if (dist && !beyond) {
                    float s = key == FILTER_NONE ? INFINITY : filter_key_distance(key);
                    if (s == 0.0f) s = dot_distance<M>(f.tables, f.codes + n * M, f.centers + (size_t)k * M);     // the sign of a zero
                    dist[n] = s;
                }
            }
        }
        if (misc[1]) break;
        if (tid == 0) misc[2] = misc[3] = 0u;                    // for the next codes, behind a barrier
    }
    wait_vector_loads();                                         // nothing may land in LDS after the workgroup has ended
}

// MARKS: the scan behind looks for single codes that are left.  Decided at run time it cost seven more spilled scalars and 0.7 of 114 us where the scan
// behind takes all codes or none (M = 16, N = 250007, K = 999).
template <int M, int CT, bool MARKS>
__global__ __launch_bounds__(512) void assign_dot_kernel(DotIn f, int32_t* __restrict__ assign, float* __restrict__ dist)
{
    __shared__ float4 tab[4096];
    __shared__ float lost_s[M * L];
    __shared__ float4 buf[2 * DOT_CHUNK / 16];
    __shared__ unsigned long long key_s[512];
    __shared__ uint32_t list_s[DOT_LIST], over_s[DOT_OVER];
    __shared__ float4 code_s[256 * CT * M / 16];
    __shared__ uint32_t misc[4];                                 // -, stop, pairs listed, codes that need all centers
    // one thread looks for all: another workgroup may set the word at any time
    if (threadIdx.x == 0) {
        misc[2] = misc[3] = 0u;
        misc[1] = __hip_atomic_load(&f.state->left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (misc[1]) return;
    if (dot_dims<M>(f.st) == 128)
        dot_scan<M, 128, CT, MARKS>(f, assign, dist, tab, lost_s, reinterpret_cast<char*>(buf), key_s, list_s, over_s, reinterpret_cast<uint32_t*>(code_s), misc);
    else
        dot_scan<M, 256, 1, MARKS>(f, assign, dist, tab, lost_s, reinterpret_cast<char*>(buf), key_s, list_s, over_s, reinterpret_cast<uint32_t*>(code_s), misc);
}

}  // namespace pqkm
