// C ABI of the PQk-means iteration for gfx950: argument validation, workspace carving and
// kernel launches.  Every entry point is declared and documented in include/pqkm.h.
#include "pqkm.h"
#include "pqkm_tuning.h"

#include <hip/hip_runtime.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <vector>

#include "pqkm_kernels.h"
#include "pqkm_filter.h"
#include "pqkm_dot.h"

// Scratch of pqkm_assign_noalloc: one array per GPU, held from the moment the library is loaded on it until the
// process ends.  In host code this name is only a handle for hipGetSymbolAddress, never an address to pass on.
static __device__ __align__(256) unsigned char scratch[PQKM_NOALLOC_SCRATCH_BYTES];

namespace {

using namespace pqkm;

// ------------------------------------------------------------------ options and profiling state
struct Options {
    int assign_kernel = 0;   // 0 auto, 1 generic, 2 tiled
    int scan_variant = 0;    // 0 auto, else a specific instantiation (tuning)
    int hist_kernel = 0;     // 0 auto, 1 global atomics, 2 LDS-privatised owner path, 3 sorted by cluster
    int profile = 0;         // bit 0: bracket scan kernels with events, bit 1: bracket whole assignment steps
    int64_t launch_codes = (int64_t)1 << 26;   // codes per scan launch
    int rounds_per_launch = 1;                 // big scans: rounds of workgroups per kernel launch, 0 = all in one
};
Options g_opt;
std::mutex g_mu;
constexpr int HIST_GROUPS = 64;        // target number of cluster groups of the LDS-privatised histogram (measured best)

// Every entry point reads the process-wide options once, here, and passes the copy down: a call never sees a
// change that another thread makes while it runs.
Options options_snapshot()
{
    std::lock_guard<std::mutex> lk(g_mu);
    return g_opt;
}

struct EventPair { hipEvent_t a, b; };
struct EventLog {
    std::vector<EventPair> pool;    // all events ever created
    size_t used = 0;                // pairs recorded since the last read
    int64_t kernels = 0;            // kernel launches inside those pairs (scan log only)
};
EventLog g_scan_log, g_step_log;    // around the scan kernels of a stretch of codes / around every whole assignment step
// scan kernels launched by this thread since it was last cleared: a stretch of codes is one launch, or one launch
// per round of workgroups
thread_local int64_t t_scan_kernels = 0;

// start of a bracket: takes (or creates) a pair and records its first event; false if none could be had
bool log_begin(EventLog& log, hipStream_t st, EventPair* ev)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (log.used == log.pool.size()) {
            EventPair e{};
            if (hipEventCreate(&e.a) == hipSuccess && hipEventCreate(&e.b) == hipSuccess) log.pool.push_back(e);
        }
        if (log.used == log.pool.size()) return false;
        *ev = log.pool[log.used++];
    }
    hipEventRecord(ev->a, st);
    return true;
}

pqkm_status log_read(EventLog& log, double* total_ms, int64_t* count)
{
    if (!total_ms || !count) return PQKM_ERR_NULL;
    std::lock_guard<std::mutex> lk(g_mu);
    double tot = 0.0;
    for (size_t i = 0; i < log.used; ++i) {
        if (hipEventSynchronize(log.pool[i].b) != hipSuccess) return PQKM_ERR_DEVICE;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, log.pool[i].a, log.pool[i].b) != hipSuccess) return PQKM_ERR_DEVICE;
        tot += ms;
    }
    *total_ms = tot;
    *count = log.kernels ? log.kernels : (int64_t)log.used;
    log.used = 0;
    log.kernels = 0;
    return PQKM_OK;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
inline bool tiled_M(int M) { return M == 4 || M == 8 || M == 16 || M == 32; }
inline bool dot_M(int M) { return M == 8 || M == 16 || M == 32; }      // has the scan on the matrix cores

struct Carve {
    size_t img_off, img_bytes, hist_off, hist_bytes, counts_off, counts_bytes, parts_off, parts_bytes, gid_off,
        gid_bytes, gco_off, plan_off, rows_off, gc8_off, plan8_off, sidx_off, seg_off, pool_off, bseg_off, skew_off,
        rank_off, tabt_off, rowoff_off, state_off, side_off, dot_off, total;
};

// room of the M = 8 lower-bound scan for what lasts from one iteration to the next (FilterSide)
inline size_t filter_side_bytes(int M, int K) { return 4096 + 512 + 2 * align256((size_t)K * M); }

// The regrouped copy of the codes (M = 4 scan) covers one scan launch of at most this many codes.
constexpr int64_t GROUP_CHUNK_MAX = (int64_t)1 << 26;
inline int64_t group_alloc(int64_t n) { return (n + 30) & ~(int64_t)15; }  // regrouped positions for n codes
constexpr int SW_C_MAX = 256 * 16;          // most codes a workgroup of the sliding-window scan takes
inline int64_t sw_alloc(int64_t n) { return ((n + SW_C_MAX - 1) / SW_C_MAX + 1) * SW_C_MAX; }   // whole workgroups of any shape

int cu_count();

// Shape of the LDS-privatised histogram pass: KT clusters per workgroup, `groups` cluster groups, S code slices.
struct HistPlan { int KT; int64_t groups; int S; bool cheap; };

HistPlan hist_plan(int64_t N, int M, int K)
{
    HistPlan p{};
    const int kt_max = (HIST_LDS_WORDS / L) / M;           // 128 KB of LDS / (M KB per cluster)
    if (kt_max < 1) return p;
    // about HIST_GROUPS groups (a byte names at most 255), within the LDS budget
    const int hg = HIST_GROUPS;
    int kt = (K + hg - 1) / hg;
    if (kt > kt_max) kt = kt_max;
    p.KT = kt;
    p.groups = ((int64_t)K + p.KT - 1) / p.KT;
    p.S = 1;
    while (p.groups * p.S < 192 && p.S < 16 && N / (2 * p.S) >= 8192) p.S *= 2;
    // every cluster group streams one byte per code: worth it while the groups fit a byte and that stays small
    p.cheap = p.groups <= 255 && (double)p.groups * (double)N <= 2.0e9;
    return p;
}

// Where the owner path is possible but the sorted one faster (nothing forced, no records from the scan, not by subspace): every
// cluster group streams a byte per code, tight clusters meet on few counters, and a heavy cluster is one workgroup's work.  Whole
// update, owner / sorted, us.  Codes without a pattern, clusters of even size: M = 2: 150 / 157 at N = 2e6, K = 8000 (the only M at
// which any was slower, up to 9 %); M = 4: 230 / 192 at 2e6, 5000; M = 8: 179 / 176 at 1e6, 4000, 214 / 202 at 3e6, 2000; M = 16: 241 /
// 198 at 3e6, 1000; M = 24: 251 / 245 at 1e6, 1200; M = 48: 250 / 204 at 1e6, 500.  Uneven clusters: 640 / 165, 598 / 171, 788 / 181,
// 1187 / 210, 2052 / 214, 1975 / 240, 3254 / 227.  Tight ones: M = 4: 355 / 164; M = 8: 415 / 159; M = 16: 1076 / 222.
// Sorted by group, which came later, it pays from 1e5 codes on where the owner path's workgroups need a second round (it then leaves half of the
// last one idle) and, in one round, where 64 KB of counters divide by M: from 12000 histograms of a subspace on at M = 4 and 8, 8000 at M =
// 16, 4800 at M = 32 and 64.  Clusters of even / of uneven size (the cube of a random number), owner : sorted.  Two rounds: M = 4, K = 3000: 49.7 :
// 39.6 / 50.9 : 41.2 at 1e5, 143 : 110 / 150 : 123 at 2e6; M = 8, 1500: 61 : 50 / 65 : 56 at 1e5; M = 12, 1333: 169 : 137 / 163 : 150 at 1e6; M = 24,
// 333: 98 : 85 / 91 : 97 at 4e5; M = 40, 400: 101 : 90 / 108 : 108 at 1e5.  One round: M = 4, K = 4000: 44.5 : 45.1 / 46.0 : 46.9 at 1e5, 102 : 92 / 117 :
// 107 at 1e6; K = 2000: 37.8 : 36.0 / 40.0 : 37.5 at 1e5, but 53.8 : 56.4 / 59.4 : 61.8 at 4e5; M = 8, K = 1000: 53.3 : 52.3 / 60.3 : 60.1 at 2e5, but 63.4 :
// 62.2 / 67.8 : 71.3 at 4e5; M = 16, K = 500: 53.5 : 51.0 / 60.3 : 60.3 at 1e5; K = 300: 98.8 : 94.0 / 133 : 105 at 1e6, but 52.7 : 54.5 / 57.9 : 59.7 at
// 1e5; M = 32, K = 150: 65.5 : 65.6 / 69.7 : 69.7 at 1e5.  Not where M leaves counters unused: M = 12, K = 1000: 65.0 : 71.4 / 74.1 : 77.9 at 2e5, K = 2000:
// 56.4 : 66.7 at 1e5; M = 24, 200: 60.4 : 65.3; M = 48, 500: 89.5 : 97.2; M = 20 (K = 400: 94 : 88 / 94 : 104 at 4e5); nor where one round without slices
// has little to do: M = 8, K = 4060: 73 : 77 / 79 : 83 at 2e5, M = 16, K = 1737: 94 : 97 at 2.2e5, but M = 32, K = 805: 144 : 138 at 3e5.  A power law gains
// more (M = 16, K = 1000, 1e6: 599 : 138).  Not in the fits whose lower-bound scans keep their keys in the sorted indices' room (`keys`).
inline bool sorted_histogram_pays(const HistPlan& hp, int64_t N, int M, int K, bool keys)
{
    if (N > (int64_t)0xffffffff) return false;
    const bool two_rounds = hp.groups * hp.S > cu_count();
    if (!keys && N >= 100000 && (M == 4 || M == 12 || (M % 8 == 0 && M != 56)) && (two_rounds || hp.S > 1 || N * M >= 4000000)) {
        const int64_t bins = (int64_t)K * M;
        if (bins >= 6000 && two_rounds) return true;
        if (M <= 8 && (bins >= 12000 || (bins >= 8000 && (N < 300000 || N >= 1500000)))) return true;
        if (M == 16 && bins >= (N >= 800000 ? 4800 : 8000)) return true;
        if ((M == 32 || M == 64) && bins >= 4800) return true;
    }
    return hp.groups > 100 && (double)hp.groups * (double)N > 2.2e8;
}

// are a fit's lower-bound scans of the kind that keeps keys by position of a code?
inline bool scans_keep_keys(int M) { return M == 4 || M == 8; }

// does the histogram take the LDS-privatised owner path for this problem (and the call's options)?
bool owner_histogram(const HistPlan& hp, int force)
{
    return hp.KT >= 1 && hp.groups <= 255 && force != 1 && force != 3 && (force == 2 || hp.cheap);
}

// The scan on the matrix cores, inside the images' room: fragments of the centers, halves of the points (all columns, and the
// first half of them), what rounding took of each, statistics.
struct DotCarve { size_t img_off, emb_off, lost_off, stat_off, check_off, total; };

DotCarve dot_carve(int M, int K)
{
    DotCarve c{};
    size_t off = 0;
    c.img_off = off;    off += align256((((size_t)K + DOT_TILE - 1) / DOT_TILE) * DOT_CHUNK);     // 256 dimensions: a chunk per tile
    c.emb_off = off;    off += (size_t)L * (256 + 128) * 2;
    c.lost_off = off;   off += (size_t)M * L * sizeof(float);
    c.stat_off = off;   off += align256((size_t)M * sizeof(DotStat));
    c.check_off = off;  off += align256((size_t)M * DOT_PARTS * sizeof(DotCheck));
    c.total = off;
    return c;
}

Carve carve(int64_t N, int M, int K)
{
    Carve c{};
    size_t off = 0;
    c.img_off = off;
    if (tiled_M(M)) {
        int TK = 128 / M;
        size_t ntiles = ((size_t)K + TK - 1) / TK;
        c.img_bytes = ntiles * (size_t)TILE_BYTES;
        // the sliding-window scan of the wide codes tiles the centers 16 at a time (M planes of 16 KB per tile)
        if (M >= 16) {
            const size_t wide = (((size_t)K + 15) / 16) * (size_t)M * 16384;
            if (wide > c.img_bytes) c.img_bytes = wide;
        }
    }
    off += align256(c.img_bytes);
    c.hist_off = off;
    c.hist_bytes = (size_t)K * M * L * sizeof(uint32_t);
    off += align256(c.hist_bytes);
    c.counts_off = off;
    c.counts_bytes = (size_t)K * sizeof(uint32_t);
    off += align256(c.counts_bytes);
    c.parts_off = off;
    HistPlan hp = hist_plan(N, M, K);
    c.parts_bytes = (hp.KT >= 1 && hp.S > 1) ? (size_t)hp.S * align256(c.hist_bytes) : 0;
    off += c.parts_bytes;
    c.gid_off = off;
    c.gid_bytes = (hp.KT >= 1 && hp.groups <= 255) ? (size_t)N : 0;
    off += align256(c.gid_bytes);
    c.gco_off = c.plan_off = c.rows_off = off;
    if (M == 4) {
        c.rows_off = off;                    // second copy of the tile images, read by the half-plane scan's epilogue
        off += align256(c.img_bytes);
        const int64_t na = group_alloc(N < GROUP_CHUNK_MAX ? N : GROUP_CHUNK_MAX);
        c.gco_off = off;
        off += align256((size_t)na * sizeof(uint2));
        c.plan_off = off;
        off += align256(sizeof(GroupPlan));
        // records the scan files by cluster group for the histogram (one scan launch, owner-path sizes only): every
        // scan workgroup owns as many records as it has code positions (at most 4096); one segment per (group, workgroup)
        c.pool_off = c.bseg_off = off;
        if (hp.KT >= 1 && hp.groups <= 255 && N <= GROUP_CHUNK_MAX - 16384) {
            c.pool_off = off;
            off += align256((size_t)(na + 4096) * sizeof(uint2));
            c.bseg_off = off;
            off += align256((size_t)hp.groups * (size_t)(na / 2048 + 2) * sizeof(uint2));
        }
    }
    // sorted-path histogram: code indices sorted by cluster (u32), every code's rank inside its cluster left by the scan
    // (pqkm_fit), cluster sizes, starts and cursors
    c.sidx_off = c.seg_off = c.state_off = off;
    if (N <= (int64_t)0xffffffff) {
        c.sidx_off = off;
        off += align256((size_t)N * sizeof(uint32_t));
        c.rank_off = off;
        off += align256((size_t)N * sizeof(uint32_t));
        c.seg_off = off;
        off += 3 * align256(((size_t)K + 1) * sizeof(uint32_t));
    }
    // keys of the lower-bound scans (8 bytes per code position of a launch): they live only while a scan runs.  Where the
    // histogram of a fused iteration takes the owner path no ranks are handed over, and the keys share the room of the
    // sorted path (the at most 30 padding positions reach into the cluster sizes, which are written after the scan).
    if (tiled_M(M)) {
        if (hp.cheap && N <= GROUP_CHUNK_MAX) {
            c.state_off = c.sidx_off;
        } else {
            c.state_off = off;
            off += align256((size_t)group_alloc(N < GROUP_CHUNK_MAX ? N : GROUP_CHUNK_MAX) * sizeof(uint64_t));
        }
    }
    c.gc8_off = c.plan8_off = off;
    if (M == 8) {
        const int64_t na = group_alloc(N < GROUP_CHUNK_MAX ? N : GROUP_CHUNK_MAX);
        c.gc8_off = off;
        off += align256((size_t)na * sizeof(uint4));
        c.plan8_off = off;
        off += align256(sizeof(GroupPlan8));
    }
    // table-built tiles (M = 4): transposed tables with a row of +inf, row offsets of the centers per tile and plane
    c.tabt_off = c.rowoff_off = off;
    if (M == 4) {
        c.tabt_off = off;
        off += align256(((size_t)M * L + 1) * L * sizeof(float));
        c.rowoff_off = off;
        off += align256((((size_t)K + 31) / 32) * 128 * sizeof(uint32_t));
    }
    // subcode words of the sliding-window scan (M = 16, 32): M/4 + 1 words per code position of one launch
    c.skew_off = off;
    if (M == 16 || M == 32) {
        const int64_t na = sw_alloc(N < GROUP_CHUNK_MAX ? N : GROUP_CHUNK_MAX);
        off += align256((size_t)na * (size_t)(M / 4 + 1) * sizeof(uint32_t));
    }
    // the side room of the M = 8 lower-bound scan, unless a problem that pqkm_assign_noalloc can hold would not fit any more (it
    // then runs the plain scans)
    c.side_off = 0;
    if (M == 8 && !(off <= PQKM_NOALLOC_SCRATCH_BYTES && off + filter_side_bytes(M, K) > PQKM_NOALLOC_SCRATCH_BYTES)) {
        c.side_off = off;
        off += filter_side_bytes(M, K);
    }
    // state of the scan on the matrix cores (DotState), under the same condition; its other arrays share the images' room
    c.dot_off = 0;
    if (dot_M(M) && !(off <= PQKM_NOALLOC_SCRATCH_BYTES && off + 256 > PQKM_NOALLOC_SCRATCH_BYTES) &&
        dot_carve(M, K).total <= c.img_bytes) {
        c.dot_off = off;
        off += 256;
    }
    c.total = off;
    return c;
}

bool shape_ok(int64_t N, int M, int K) { return N >= 0 && K >= 1 && M >= 1 && M <= 64; }

pqkm_status check_device()
{
    static thread_local int checked_dev = -1;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return PQKM_ERR_DEVICE;
    if (dev == checked_dev) return PQKM_OK;
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, dev) != hipSuccess) return PQKM_ERR_DEVICE;
    if (strncmp(p.gcnArchName, "gfx950", 6) != 0) return PQKM_ERR_DEVICE;
    checked_dev = dev;
    return PQKM_OK;
}

// Device address of `scratch` on the current device: asked of the runtime once per device (each GPU holds its own
// copy at its own address) and kept.
constexpr int SCRATCH_MAX_DEVICES = 64;
void* g_scratch_ptr[SCRATCH_MAX_DEVICES];
std::mutex g_scratch_mu;

pqkm_status scratch_of_current_device(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= SCRATCH_MAX_DEVICES) return PQKM_ERR_DEVICE;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PQKM_ERR_DEVICE;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return PQKM_OK;
}

pqkm_status launched()
{
    return hipGetLastError() == hipSuccess ? PQKM_OK : PQKM_ERR_DEVICE;
}

pqkm_status check_workspace(const void* ws, size_t bytes, size_t need)
{
    if (need == 0) return PQKM_OK;
    if (ws == nullptr || ((uintptr_t)ws & 255) != 0 || bytes < need) return PQKM_ERR_WORKSPACE;
    return PQKM_OK;
}

// compute units of the current device (asked once; 256 if the query fails)
int cu_count()
{
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1)
            v = 256;
        return v;
    }();
    return n;
}

// ------------------------------------------------------------------ scan launch
template <int M, int R, int THREADS, bool PF>
void launch_scan(const uint8_t* codes, int64_t N, const float4* img, int ntiles, int32_t* assign, float* dist,
                 hipStream_t st)
{
    using S = ScanShape<M>;
    constexpr int C = (THREADS / S::LPS) * R;
    int64_t nwg = (N + C - 1) / C;
    hipLaunchKernelGGL((assign_scan_kernel<M, R, THREADS, PF>), dim3((unsigned)nwg), dim3(THREADS), 0, st, codes, N,
                       img, ntiles, assign, dist);
}

template <int R, int THREADS>
void launch_scan4s(const uint8_t* codes, int64_t N, const float4* img, int ntiles, int32_t* assign, float* dist,
                   hipStream_t st)
{
    constexpr int C = (THREADS / 4) * R;
    int64_t nwg = (N + C - 1) / C;
    hipLaunchKernelGGL((assign_scan4s_kernel<R, THREADS>), dim3((unsigned)nwg), dim3(THREADS), 0, st, codes, N, img,
                       ntiles, assign, dist);
}

template <int R, int THREADS, int DEPTH, bool BUCKET = false>
void launch_scan4p(const uint8_t* codes, int64_t N, const uint2* gco, const float4* img, const float4* rows,
                   int ntiles, int32_t* assign, float* dist, hipStream_t st, BucketOut bo = BucketOut{},
                   RankOut ro = RankOut{})
{
    constexpr int C = (THREADS / 4) * R;
    int64_t nwg = (N + C - 1) / C;
    hipLaunchKernelGGL((assign_scan4p_kernel<R, THREADS, DEPTH, BUCKET>), dim3((unsigned)nwg), dim3(THREADS), 0, st, codes,
                       N, gco, img, rows, ntiles, assign, dist, bo, ro);
}

template <int M, int R, int THREADS, int DEPTH = 1>
void launch_scan_skew(const uint8_t* codes, int64_t N, const float4* img, int ntiles, int32_t* assign, float* dist,
                      hipStream_t st, const uint32_t* only_if)
{
    constexpr int C = (THREADS / (128 / M / 4)) * R;
    int64_t nwg = (N + C - 1) / C;
    hipLaunchKernelGGL((assign_scan_skew_kernel<M, R, THREADS, DEPTH>), dim3((unsigned)nwg), dim3(THREADS), 0, st, codes,
                       N, img, ntiles, assign, dist, only_if);
}

// tile image layout a scan shape reads: 0 = [m][x][k], 1 = [x][m][k] (subspace-skewed scans), 2 = half planes
// (variant 0, the default for M = 4, regroups the codes and runs the half-plane scan; variant 34 is the
// subspace-skewed scan, which needs no regrouping and is used for few centers or few codes)
inline int variant_layout(int M, int variant)
{
    if (M == 4) {
        if ((variant >= 40 && variant <= 49) || (variant >= 70 && variant <= 99)) return 2;
        return (variant >= 30 && variant <= 39) ? 1 : 0;
    }
    if (M == 8 && ((variant >= 40 && variant <= 49) || (variant >= 70 && variant <= 84))) return 0;   // [m][x][k]
    return variant != 1 ? 1 : 0;  // M = 8, 16, 32: every other shape but 1 (the unskewed tiled scan) is skewed
}

template <int R, int THREADS, int DEPTH>
void launch_scan8p(const uint8_t* codes, int64_t N, const uint4* gc8, const float4* img, int ntiles, int32_t* assign,
                   float* dist, hipStream_t st, RankOut ro = RankOut{}, int rounds_per_launch = 0)
{
    constexpr int C = (THREADS / 4) * R;
    int64_t nwg = (N + C - 1) / C;
    if (gc8 && rounds_per_launch > 0) {
        // regrouped codes, results go to the codes' original positions: any stretch of workgroups can be a launch
        // of its own, and the workgroups of a launch start in step (see launch_scan4q_rounds)
        const int64_t per = (int64_t)rounds_per_launch * cu_count();
        for (int64_t w0 = 0; w0 < nwg; w0 += per) {
            const int64_t cnt = nwg - w0 < per ? nwg - w0 : per;
            hipLaunchKernelGGL((assign_scan8p_kernel<R, THREADS, DEPTH>), dim3((unsigned)cnt), dim3(THREADS), 0, st, codes,
                               N - w0 * C, gc8 + w0 * C, img, ntiles, assign, dist, ro);
            ++t_scan_kernels;
        }
        return;
    }
    hipLaunchKernelGGL((assign_scan8p_kernel<R, THREADS, DEPTH>), dim3((unsigned)nwg), dim3(THREADS), 0, st, codes, N,
                       gc8, img, ntiles, assign, dist, ro);
}

template <int M>
void launch_scan_M(int variant, const uint8_t* codes, int64_t N, const float4* img, const float4* rows, int ntiles,
                   int32_t* assign, float* dist, hipStream_t st, const uint32_t* only_if);

// Sliding-window scan of the wide codes (variants 50..59): the subcode words of this launch, then the scan.
// Shapes: 512 threads with 16 or 8 codes per lane-slot (4096 or 2048 codes per workgroup, variants 51 and 52) and
// 1024 threads with 6 (3072 codes, variant 53); variant 50 chooses by the number of rounds: a round costs about
// R + 5.5 with 512 threads (R codes' reads per phase, a 64 KB fill worth 4 and two barriers) and, measured, 0.73 of
// the 16-code round with 1024 threads (16.3 ms against 11.9 ms per round at M = 32, K = 1e4).
struct SwShape { int R, threads; };
inline SwShape sw_shape(int variant, int64_t n)
{
    if (variant == 51) return {16, 512};
    if (variant == 52) return {8, 512};
    if (variant == 53) return {6, 1024};
    const int ncu = cu_count();
    static const SwShape cand[] = {{16, 512}, {6, 1024}, {8, 512}};
    static const double round_cost[] = {21.5, 15.7, 13.5};
    SwShape best = cand[0];
    double best_cost = 1e300;
    for (int i = 0; i < 3; ++i) {
        const int64_t C = (int64_t)(cand[i].threads / 2) * cand[i].R;
        const int64_t wgs = (n + C - 1) / C;
        const double cost = (double)((wgs + ncu - 1) / ncu) * round_cost[i];
        if (cost < best_cost) { best_cost = cost; best = cand[i]; }
    }
    return best;
}

template <int M>
pqkm_status launch_scan_sw(int variant, const uint8_t* codes, int64_t N, uint32_t* S, const float4* img, int ntiles16,
                           int32_t* assign, float* dist, hipStream_t st, RankOut ro, int rounds_per_launch, const uint32_t* only_if)
{
    const SwShape sh = sw_shape(variant, N);
    const bool wide = sh.threads == 1024;
    const int R = sh.R;
    const int64_t C = (int64_t)(sh.threads / 2) * R;
    const int64_t nwg = (N + C - 1) / C;
    const int64_t n_alloc = nwg * C;
    hipLaunchKernelGGL((code_skew_kernel<M>), dim3((unsigned)((n_alloc + 255) / 256)), dim3(256), 0, st, codes, N, S,
                       n_alloc, only_if);
    // kernel launches of rounds_per_launch rounds of workgroups each, so that the workgroups start in step again
    // (see launch_scan4q_rounds)
    const int64_t per = rounds_per_launch > 0 ? (int64_t)rounds_per_launch * cu_count() : nwg;
    for (int64_t w0 = 0; w0 < nwg; w0 += per) {
        const int64_t cnt = nwg - w0 < per ? nwg - w0 : per;
        if (wide)
            hipLaunchKernelGGL((assign_scan_sw_kernel<M, 6, 1024, 2>), dim3((unsigned)cnt), dim3(1024), 0, st, codes, N, S,
                               n_alloc, img, ntiles16, assign, dist, ro, w0, only_if);
        else if (R == 8)
            hipLaunchKernelGGL((assign_scan_sw_kernel<M, 8, 512, 3>), dim3((unsigned)cnt), dim3(512), 0, st, codes, N, S,
                               n_alloc, img, ntiles16, assign, dist, ro, w0, only_if);
        else
            hipLaunchKernelGGL((assign_scan_sw_kernel<M, 16, 512, 2>), dim3((unsigned)cnt), dim3(512), 0, st, codes, N, S,
                               n_alloc, img, ntiles16, assign, dist, ro, w0, only_if);
        ++t_scan_kernels;
    }
    return launched();
}

// M = 4 scans over regrouped codes: variants 70..79

// Codes per lane-slot R of the 512-thread half-plane scan (a workgroup takes 128 R codes, one workgroup per
// compute unit at a time).  The time of a launch is about rounds * (R + 7) with rounds = ceil(workgroups / CUs):
// R codes' reads per tile plus a fill and two barriers worth about 7.  Below a few rounds the rounding decides:
// 1.1e6 codes are 269 workgroups at R = 32, two rounds, but 430 at R = 20, two rounds of 5/8 the length.
int scan4p_codes_per_slot(int64_t n_alloc)
{
    const int ncu = cu_count();
    static const int cand[] = {32, 31, 28, 24, 20, 16};
    int best = 32;
    int64_t best_cost = INT64_MAX;
    for (int R : cand) {
        const int64_t wgs = (n_alloc + 128 * R - 1) / (128 * R);
        const int64_t cost = ((wgs + ncu - 1) / ncu) * (R + 7);
        if (cost < best_cost) { best_cost = cost; best = R; }
    }
    return best;
}

// bo != nullptr: the scan also files (code, center) records by cluster group for the histogram pass (variant 70
// only); *nwg_out receives the number of scan workgroups = the row length of the segment table
void launch_scan_grouped(int variant, const uint2* gco, int64_t n_alloc, const float4* img, const float4* rows,
                         int ntiles, int32_t* assign, float* dist, hipStream_t st, const BucketOut* bo = nullptr,
                         int* nwg_out = nullptr, RankOut ro = RankOut{})
{
    int R = 0;
    switch (variant) {
        case 70: R = scan4p_codes_per_slot(n_alloc); break;
        case 71: R = 28; break;
        case 72: R = 31; break;
        case 73: launch_scan4p<16, 1024, 1>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, BucketOut{}, ro); return;
        case 74: R = 24; break;
        case 75: R = 20; break;
        case 76: R = 16; break;
        default: R = 32; break;      // 77..79
    }
    if (bo) {
        if (nwg_out) *nwg_out = (int)((n_alloc + 128 * R - 1) / (128 * R));
        switch (R) {
            case 16: launch_scan4p<16, 512, 3, true>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, *bo); break;
            case 20: launch_scan4p<20, 512, 3, true>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, *bo); break;
            case 24: launch_scan4p<24, 512, 3, true>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, *bo); break;
            case 28: launch_scan4p<28, 512, 3, true>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, *bo); break;
            case 31: launch_scan4p<31, 512, 3, true>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, *bo); break;
            default: launch_scan4p<32, 512, 3, true>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, *bo); break;
        }
        return;
    }
    switch (R) {
        case 16: launch_scan4p<16, 512, 3>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, BucketOut{}, ro); break;
        case 20: launch_scan4p<20, 512, 3>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, BucketOut{}, ro); break;
        case 24: launch_scan4p<24, 512, 3>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, BucketOut{}, ro); break;
        case 28: launch_scan4p<28, 512, 3>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, BucketOut{}, ro); break;
        case 31: launch_scan4p<31, 512, 3>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, BucketOut{}, ro); break;
        default: launch_scan4p<32, 512, 3>(nullptr, n_alloc, gco, img, rows, ntiles, assign, dist, st, BucketOut{}, ro); break;
    }
}

// M = 4 scan over regrouped codes with two-lane slots (256 R codes per workgroup): variants 80..89
int scan4q_codes_per_slot(int variant, int64_t n_alloc)
{
    // (32 and 30 codes per lane-slot spill registers inside the tile loop: 0.49 and 0.61 of the LDS peak against 0.72)
    switch (variant) {
        case 81: return 26;
        case 82: return 28;
        case 83: return 24;
        case 84: return 16;
        default: break;
    }
    const int ncu = cu_count();
    static const int cand[] = {28, 26, 24, 16};
    int best = 28;
    int64_t best_cost = INT64_MAX;
    for (int R : cand) {
        const int64_t wgs = (n_alloc + 256 * R - 1) / (256 * R);
        const int64_t cost = ((wgs + ncu - 1) / ncu) * (2 * R + 13);      // 512 R clocks of reads per tile, about 3.3k of fill and barriers
        if (cost < best_cost) { best_cost = cost; best = R; }
    }
    return best;
}

template <int R>
void launch_scan4q_rounds(const uint2* gco, int64_t n_alloc, const float4* img, const float4* rows, int ntiles,
                          int32_t* assign, float* dist, hipStream_t st, RankOut ro, int rounds_per_launch)
{
    // The workgroups of a kernel launch start together and walk the tile images in step, so that a tile is fetched
    // from memory once per XCD and then served from its L2; over many rounds of workgroups they drift apart.  With
    // rounds_per_launch > 0 the codes are issued in kernel launches of that many rounds, each starting in step again.
    constexpr int64_t C = 256 * (int64_t)R;
    const int64_t nwg = (n_alloc + C - 1) / C;
    const int64_t per = rounds_per_launch > 0 ? (int64_t)rounds_per_launch * cu_count() : nwg;
    for (int64_t w0 = 0; w0 < nwg; w0 += per) {
        const int64_t cnt = nwg - w0 < per ? nwg - w0 : per;
        hipLaunchKernelGGL((assign_scan4q_kernel<R, 512, 2>), dim3((unsigned)cnt), dim3(512), 0, st, n_alloc - w0 * C,
                           gco + w0 * C, img, rows, ntiles, assign, dist, ro, TileSource{});
        ++t_scan_kernels;
    }
}

void launch_scan_grouped_q(int variant, const uint2* gco, int64_t n_alloc, const float4* img, const float4* rows,
                           int ntiles, int32_t* assign, float* dist, hipStream_t st, RankOut ro, TileSource ts,
                           int rounds_per_launch)
{
    const int R = scan4q_codes_per_slot(variant >= 90 ? variant - 10 : variant, n_alloc);
    const int64_t nwg = (n_alloc + 256 * (int64_t)R - 1) / (256 * (int64_t)R);
    if (ts.tabT) {
        switch (R) {
            case 16:
                hipLaunchKernelGGL((assign_scan4q_kernel<16, 512, 2, true>), dim3((unsigned)nwg), dim3(512), 0, st, n_alloc,
                                   gco, img, rows, ntiles, assign, dist, ro, ts);
                break;
            case 24:
                hipLaunchKernelGGL((assign_scan4q_kernel<24, 512, 2, true>), dim3((unsigned)nwg), dim3(512), 0, st, n_alloc,
                                   gco, img, rows, ntiles, assign, dist, ro, ts);
                break;
            case 26:
                hipLaunchKernelGGL((assign_scan4q_kernel<26, 512, 2, true>), dim3((unsigned)nwg), dim3(512), 0, st, n_alloc,
                                   gco, img, rows, ntiles, assign, dist, ro, ts);
                break;
            default:
                hipLaunchKernelGGL((assign_scan4q_kernel<28, 512, 2, true>), dim3((unsigned)nwg), dim3(512), 0, st, n_alloc,
                                   gco, img, rows, ntiles, assign, dist, ro, ts);
                break;
        }
        return;
    }
    switch (R) {
        case 16: launch_scan4q_rounds<16>(gco, n_alloc, img, rows, ntiles, assign, dist, st, ro, rounds_per_launch); break;
        case 24: launch_scan4q_rounds<24>(gco, n_alloc, img, rows, ntiles, assign, dist, st, ro, rounds_per_launch); break;
        case 26: launch_scan4q_rounds<26>(gco, n_alloc, img, rows, ntiles, assign, dist, st, ro, rounds_per_launch); break;
        default: launch_scan4q_rounds<28>(gco, n_alloc, img, rows, ntiles, assign, dist, st, ro, rounds_per_launch); break;
    }
}

// M = 4, two-lane slots, half tiles loaded straight into LDS (variants 85..89): codes per workgroup
struct Scan4hShape { int R, threads; };
Scan4hShape scan4h_shape(int variant)
{
    switch (variant) {
        case 86: return {12, 1024};
        case 87: return {14, 1024};
        case 88: return {32, 512};
        case 89: return {8, 1024};
        default: return {16, 1024};
    }
}
inline int64_t scan4h_codes_per_workgroup(int variant)
{
    const Scan4hShape sh = scan4h_shape(variant);
    return (int64_t)(sh.threads / 2) * sh.R;
}

template <int R, int THREADS, int DEPTH>
void launch_scan4h_rounds(const uint2* gco, int64_t n_alloc, const float4* img, const float4* rows, int ntiles,
                          int nhalves, int32_t* assign, float* dist, hipStream_t st, RankOut ro, int rounds_per_launch)
{
    // one kernel launch per rounds_per_launch rounds of workgroups (see launch_scan4q_rounds)
    constexpr int64_t C = (THREADS / 2) * (int64_t)R;
    const int64_t nwg = (n_alloc + C - 1) / C;
    const int64_t per = rounds_per_launch > 0 ? (int64_t)rounds_per_launch * cu_count() : nwg;
    for (int64_t w0 = 0; w0 < nwg; w0 += per) {
        const int64_t cnt = nwg - w0 < per ? nwg - w0 : per;
        hipLaunchKernelGGL((assign_scan4h_kernel<R, THREADS, DEPTH>), dim3((unsigned)cnt), dim3(THREADS), 0, st,
                           n_alloc - w0 * C, gco + w0 * C, img, rows, ntiles, nhalves, assign, dist, ro);
        ++t_scan_kernels;
    }
}

void launch_scan_grouped_h(int variant, const uint2* gco, int64_t n_alloc, const float4* img, const float4* rows,
                           int ntiles, int nhalves, int32_t* assign, float* dist, hipStream_t st, RankOut ro,
                           int rounds_per_launch)
{
    switch (variant) {
        case 86: launch_scan4h_rounds<12, 1024, 4>(gco, n_alloc, img, rows, ntiles, nhalves, assign, dist, st, ro, rounds_per_launch); break;
        case 87: launch_scan4h_rounds<14, 1024, 3>(gco, n_alloc, img, rows, ntiles, nhalves, assign, dist, st, ro, rounds_per_launch); break;
        case 88: launch_scan4h_rounds<32, 512, 2>(gco, n_alloc, img, rows, ntiles, nhalves, assign, dist, st, ro, rounds_per_launch); break;
        case 89: launch_scan4h_rounds<8, 1024, 3>(gco, n_alloc, img, rows, ntiles, nhalves, assign, dist, st, ro, rounds_per_launch); break;
        default: launch_scan4h_rounds<16, 1024, 3>(gco, n_alloc, img, rows, ntiles, nhalves, assign, dist, st, ro, rounds_per_launch); break;
    }
}

// The 4096-code shape of the LDS-direct scan, filing (code, center) records by cluster group for the histogram: all
// workgroups in one launch (a segment is named by its workgroup's index in the grid).
void launch_scan4h_bucket(const uint2* gco, int64_t n_alloc, const float4* img, const float4* rows, int ntiles,
                          int nhalves, int32_t* assign, float* dist, hipStream_t st, BucketOut bo, int* nwg_out)
{
    constexpr int64_t C = 512 * 8;
    const int64_t nwg = (n_alloc + C - 1) / C;
    hipLaunchKernelGGL((assign_scan4h_kernel<8, 1024, 3, true>), dim3((unsigned)nwg), dim3(1024), 0, st, n_alloc, gco, img,
                       rows, ntiles, nhalves, assign, dist, RankOut{}, bo);
    ++t_scan_kernels;
    *nwg_out = (int)nwg;
}

// M = 4, many codes: the four-lane scan (variant 70) or one of the shapes of the LDS-direct scan (85..87, 89), by the time
// the rounds of workgroups take.  Clocks per tile and workgroup of C codes, from the measured times: four lanes per
// code 2.30 C + 2065 (the fill of 128 KB between two barriers), LDS-direct 2.45 C + 1064 (two halves).
int choose_scan4_large(int64_t n, double* clocks = nullptr)
{
    const int ncu = cu_count();
    const int64_t na = group_alloc(n);
    auto rounds = [&](int64_t C) { return ((na + C - 1) / C + ncu - 1) / ncu; };
    const int64_t c4p = 128 * (int64_t)scan4p_codes_per_slot(na);
    double best_cost = (double)rounds(c4p) * (2.30 * (double)c4p + 2065.0);
    int best = 70;
    if (n >= ((int64_t)1 << 23)) {                     // stretches are cut to whole rounds of the largest shape
        if (clocks) *clocks = (double)rounds(8192) * (2.45 * 8192.0 + 1064.0);
        return 85;
    }
    static const int cand[] = {85, 87, 86, 89};
    for (int v : cand) {
        const int64_t C = scan4h_codes_per_workgroup(v);
        const double cost = (double)rounds(C) * (2.45 * (double)C + 1064.0);
        if (cost < best_cost) { best_cost = cost; best = v; }
    }
    if (clocks) *clocks = best_cost;
    return best;
}

// M = 4 scan through lower bounds (variants 60..64): codes per workgroup 512 R
// Fewest centers, by iteration of a call.  What a code costs beside the scan of its tiles is candidates, four table lines
// through the L2 each: several in the first iteration, less from the bound that the center of the iteration before gives,
// less still once most centers no longer change.  Measured against the plain scans, ms per iteration, N = 1e6: first
// 0.28 / 0.24 at K = 1000, 0.337 / 0.313 at 1500; second and third 0.181 / 0.180 at K = 700, 0.202 / 0.220 at 1000;
// later 0.132 / 0.172 at K = 700.  N = 3e6, K = 2500: 1.02 / 1.27, 0.84 / 1.26, 0.69 / 1.26.  Where one round of workgroups covers
// the codes there is none to warn the next ones off tables that the bounds do not separate (K = 2500, distances of one dimension:
// 2.1 times the plain scan, 1.0 over several rounds), so a first iteration needs more to gain: 0.95 at K = 2500, 0.8 at 5000.
inline int filter4_min_k(int iteration, int64_t N)
{
    return iteration == 0 ? (N > (int64_t)cu_count() * 8192 ? 2500 : 4000) : iteration < 3 ? 900 : 500;
}
int filter4_codes_per_slot(int variant, int64_t n_alloc)
{
    switch (variant) {
        case 61: return 16;
        case 62: return 12;
        case 63: return 8;
        case 64: return 4;
        default: break;
    }
    const int ncu = cu_count();
    static const int cand[] = {16, 12, 8, 4};
    int best = 16;
    double best_cost = 1e300;
    for (int R : cand) {
        const int64_t wgs = (n_alloc + 512 * R - 1) / (512 * R);
        // measured at K = 1e5 per round: 7.6, 5.9, 4.1 ms for R = 16, 12, 8
        const double cost = (double)((wgs + ncu - 1) / ncu) * (R + 1.4);
        if (cost < best_cost) { best_cost = cost; best = R; }
    }
    return best;
}

template <int M, int R, int THREADS = 1024, int DEPTH = 3>
void launch_filter_rounds(const typename FilterCode<M>::Raw* gco, int64_t n_alloc, FilterIn f, int32_t* assign, float* dist, hipStream_t st,
                           RankOut ro, int rounds_per_launch)
{
    // one kernel launch per rounds_per_launch rounds of workgroups (see launch_scan4q_rounds)
    constexpr int64_t C = THREADS / 2 * (int64_t)R;
    const int64_t nwg = (n_alloc + C - 1) / C;
    const int64_t per = rounds_per_launch > 0 ? (int64_t)rounds_per_launch * cu_count() : nwg;
    unsigned long long* state = f.state;
    for (int64_t w0 = 0; w0 < nwg; w0 += per) {
        const int64_t cnt = nwg - w0 < per ? nwg - w0 : per;
        f.state = state + w0 * C;
        f.launched = (int)w0;
        hipLaunchKernelGGL((assign_filter_kernel<M, R, THREADS, DEPTH, false>), dim3((unsigned)cnt), dim3(THREADS), 0, st, n_alloc - w0 * C,
                           gco + w0 * C, f, assign, dist, ro, BucketOut{});
        ++t_scan_kernels;
    }
}

void launch_filter4(int variant, const uint2* gco, int64_t n_alloc, const FilterIn& f, int32_t* assign, float* dist,
                    hipStream_t st, RankOut ro, int rounds_per_launch)
{
    switch (filter4_codes_per_slot(variant, n_alloc)) {
        case 4: launch_filter_rounds<4, 4>(gco, n_alloc, f, assign, dist, st, ro, rounds_per_launch); break;
        case 8: launch_filter_rounds<4, 8>(gco, n_alloc, f, assign, dist, st, ro, rounds_per_launch); break;
        case 12: launch_filter_rounds<4, 12>(gco, n_alloc, f, assign, dist, st, ro, rounds_per_launch); break;
        default: launch_filter_rounds<4, 16>(gco, n_alloc, f, assign, dist, st, ro, rounds_per_launch); break;
    }
}

// Centers from which the bound of a first iteration comes from the pair tables: K >= 400 leaves room for them (1 MB) behind
// the byte tiles in either case
constexpr int FILTER_PAIRS_MIN_K = 500;
// the same for M = 8, N = 4.2e6: first 4.2 / 4.1 at K = 1500, 5.8 / 7.3 at 4000; second and third 1.53 / 1.35 at K = 600,
// 1.94 / 2.64 at 1500; later 0.93 / 1.35 at K = 600
inline int filter8_min_k(int iteration) { return iteration == 0 ? 1800 : iteration < 3 ? 900 : 500; }

// M = 8 (variants 60..63): codes per workgroup 256 R, 512 threads (with 1024 and half the registers the loop spills)
int filter8_codes_per_slot(int variant, int64_t n_alloc)
{
    if (variant == 61) return 24;
    if (variant == 62) return 16;
    if (variant == 63) return 8;
    const int ncu = cu_count();
    static const int cand[] = {24, 16, 8};
    int best = 24;
    double best_cost = 1e300;
    for (int R : cand) {
        const int64_t wgs = (n_alloc + 256 * R - 1) / (256 * R);
        // measured at K = 1e4 per round: 1.67, 1.23, 0.77 ms for R = 24, 16, 8
        const double cost = (double)((wgs + ncu - 1) / ncu) * (R + 6.4);
        if (cost < best_cost) { best_cost = cost; best = R; }
    }
    return best;
}

void launch_filter8(int variant, const uint4* gc8, int64_t n_alloc, const FilterIn& f, int32_t* assign, float* dist,
                    hipStream_t st, RankOut ro, int rounds_per_launch)
{
    switch (filter8_codes_per_slot(variant, n_alloc)) {
        case 8: launch_filter_rounds<8, 8, 512, 4>(gc8, n_alloc, f, assign, dist, st, ro, rounds_per_launch); break;
        case 16: launch_filter_rounds<8, 16, 512, 4>(gc8, n_alloc, f, assign, dist, st, ro, rounds_per_launch); break;
        default: launch_filter_rounds<8, 24, 512, 4>(gc8, n_alloc, f, assign, dist, st, ro, rounds_per_launch); break;
    }
}

// The plain scan of what a lower-bound scan left (it ends at once if that is nothing), in the shape that the rounds favour were
// it everything: the LDS-direct scan at M = 4, the two-lane scan at M = 8.  Not counted as a scan kernel.
void launch_left4(const uint2* gco, int64_t n_alloc, const float4* img, const float4* rows, int ntiles, int nhalves,
                  const FilterIn& f, int32_t* assign, float* dist, hipStream_t st, RankOut ro, const BucketOut* bo)
{
    const int64_t ncu = cu_count();
    auto wgs = [&](int R) { return (n_alloc + 512 * R - 1) / (512 * R); };
    auto cost = [&](int R) { return (double)((wgs(R) + ncu - 1) / ncu) * (2.45 * 512 * R + 1064.0); };     // choose_scan4_large
    if (bo)
        hipLaunchKernelGGL((assign_scan4h_kernel<8, 1024, 3, true, true>), dim3((unsigned)wgs(8)), dim3(1024), 0, st, n_alloc, gco,
                           img, rows, ntiles, nhalves, assign, dist, RankOut{}, *bo, f.state);
    else if (cost(8) < cost(16))
        hipLaunchKernelGGL((assign_scan4h_kernel<8, 1024, 3, false, true>), dim3((unsigned)wgs(8)), dim3(1024), 0, st, n_alloc, gco,
                           img, rows, ntiles, nhalves, assign, dist, ro, BucketOut{}, f.state);
    else
        hipLaunchKernelGGL((assign_scan4h_kernel<16, 1024, 3, false, true>), dim3((unsigned)wgs(16)), dim3(1024), 0, st, n_alloc, gco,
                           img, rows, ntiles, nhalves, assign, dist, ro, BucketOut{}, f.state);
}

void launch_left8(const uint4* gc8, int64_t n_alloc, const float4* img, int ntiles, const FilterIn& f, int32_t* assign, float* dist,
                  hipStream_t st, RankOut ro)
{
    const int64_t ncu = cu_count();
    auto wgs = [&](int R) { return (n_alloc + 256 * R - 1) / (256 * R); };
    auto cost = [&](int R) { return ((wgs(R) + ncu - 1) / ncu) * (2 * R + 13); };                          // scan8q_codes_per_slot
    if (cost(16) < cost(24))
        hipLaunchKernelGGL((assign_scan8q_kernel<16, 512, 3, true>), dim3((unsigned)wgs(16)), dim3(512), 0, st, n_alloc, gc8, img,
                           ntiles, assign, dist, ro, f.state);
    else
        hipLaunchKernelGGL((assign_scan8q_kernel<24, 512, 2, true>), dim3((unsigned)wgs(24)), dim3(512), 0, st, n_alloc, gc8, img,
                           ntiles, assign, dist, ro, f.state);
}

// the 4096-code shape, filing (code, center) records by cluster group for the histogram: all workgroups in one launch
void launch_filter4_bucket(const uint2* gco, int64_t n_alloc, const FilterIn& f, int32_t* assign, float* dist,
                           hipStream_t st, BucketOut bo, int* nwg_out)
{
    constexpr int64_t C = 512 * 8;
    const int64_t nwg = (n_alloc + C - 1) / C;
    hipLaunchKernelGGL((assign_filter_kernel<4, 8, 1024, 3, true>), dim3((unsigned)nwg), dim3(1024), 0, st, n_alloc, gco, f, assign,
                       dist, RankOut{}, bo);
    ++t_scan_kernels;
    *nwg_out = (int)nwg;
}

// M = 8 scans over regrouped codes: variants 70..79.  Variant 70 chooses the codes per lane-slot like the M = 4
// scan does: rounds * (R + 9) with rounds = ceil(workgroups / CUs) (8e6 codes: 11 rounds of 2605 workgroups at
// R = 24, 10 rounds of 2500 at R = 25, measured 12.2 ms against 11.4 ms at K = 4000).
int scan8p_codes_per_slot(int64_t n_alloc)
{
    const int ncu = cu_count();
    static const int cand[] = {25, 24, 22, 20, 18, 16};
    int best = 24;
    int64_t best_cost = INT64_MAX;
    for (int R : cand) {
        const int64_t wgs = (n_alloc + 128 * R - 1) / (128 * R);
        const int64_t cost = ((wgs + ncu - 1) / ncu) * (R + 9);
        if (cost < best_cost) { best_cost = cost; best = R; }
    }
    return best;
}

void launch_scan_grouped8(int variant, const uint4* gc8, int64_t n_alloc, const float4* img, int ntiles, int32_t* assign,
                          float* dist, hipStream_t st, RankOut ro = RankOut{}, int rpl = 0)
{
    int R = 0;
    switch (variant) {
        case 70: R = scan8p_codes_per_slot(n_alloc); break;
        case 71: launch_scan8p<12, 1024, 2>(nullptr, n_alloc, gc8, img, ntiles, assign, dist, st, ro, rpl); return;
        case 72: launch_scan8p<16, 512, 8>(nullptr, n_alloc, gc8, img, ntiles, assign, dist, st, ro, rpl); return;
        case 73: launch_scan8p<24, 512, 2>(nullptr, n_alloc, gc8, img, ntiles, assign, dist, st, ro, rpl); return;
        case 74: R = 25; break;
        case 75: R = 22; break;
        case 76: R = 20; break;
        case 77: R = 18; break;
        case 78: R = 16; break;
        default: R = 24; break;
    }
    switch (R) {
        case 16: launch_scan8p<16, 512, 4>(nullptr, n_alloc, gc8, img, ntiles, assign, dist, st, ro, rpl); break;
        case 18: launch_scan8p<18, 512, 4>(nullptr, n_alloc, gc8, img, ntiles, assign, dist, st, ro, rpl); break;
        case 20: launch_scan8p<20, 512, 4>(nullptr, n_alloc, gc8, img, ntiles, assign, dist, st, ro, rpl); break;
        case 22: launch_scan8p<22, 512, 4>(nullptr, n_alloc, gc8, img, ntiles, assign, dist, st, ro, rpl); break;
        case 25: launch_scan8p<25, 512, 4>(nullptr, n_alloc, gc8, img, ntiles, assign, dist, st, ro, rpl); break;
        default: launch_scan8p<24, 512, 4>(nullptr, n_alloc, gc8, img, ntiles, assign, dist, st, ro, rpl); break;
    }
}

// Codes per lane-slot of the two-lane M = 8 scan (a workgroup takes 256 R codes) by the rounds, in the unit of
// scan8p_codes_per_slot (128 codes' reads per tile): 2 R + 13.  24 codes per lane-slot fit the registers with the
// reads of two steps in flight instead of three (0.692 of the LDS peak against 0.686 for 22 at whole rounds; with
// three they spill and lose 8 %); 1024 threads with 10 or 8 codes per lane-slot reach 0.65 and 0.63.
int scan8q_codes_per_slot(int64_t n_alloc, int64_t* cost_out)
{
    const int ncu = cu_count();
    static const int cand[] = {24, 22, 20, 16};
    int best = 22;
    int64_t best_cost = INT64_MAX;
    for (int r : cand) {
        const int64_t wgs = (n_alloc + 256 * r - 1) / (256 * r);
        const int64_t cost = ((wgs + ncu - 1) / ncu) * (2 * r + 13);
        if (cost < best_cost) { best_cost = cost; best = r; }
    }
    if (cost_out) *cost_out = best_cost;
    return best;
}

// M = 8, many codes: four lanes per code (variant 70) or two (80), by the time the rounds take.  Per unit the
// two-lane scan is about 5 % faster (74 against 79 us at N = 1e7, K = 1e4); with few tiles its longer epilogue shows.
int choose_scan8_large(int64_t n, int K)
{
    if (K < 512) return 70;
    const int64_t na = group_alloc(n < GROUP_CHUNK_MAX - 16384 ? n : GROUP_CHUNK_MAX - 16384);
    const int ncu = cu_count();
    const int R = scan8p_codes_per_slot(na);
    const int64_t wgs = (na + 128 * R - 1) / (128 * R);
    const int64_t cost_p = ((wgs + ncu - 1) / ncu) * (R + 9);
    int64_t cost_q = 0;
    scan8q_codes_per_slot(na, &cost_q);
    return (double)cost_q * 0.95 < (double)cost_p ? 80 : 70;
}

// M = 8 scan over regrouped codes with two-lane slots (256 R codes per workgroup): variants 80..84
template <int R, int THREADS = 512, int DEPTH = 3>
void launch_scan8q_rounds(const uint4* gc8, int64_t n_alloc, const float4* img, int ntiles, int32_t* assign,
                          float* dist, hipStream_t st, RankOut ro, int rounds_per_launch)
{
    // one kernel launch per rounds_per_launch rounds of workgroups (see launch_scan4q_rounds), 0 = one for all.
    // (While the left-over groups were spread singly, a launch per round was 4 % slower for this scan: every round
    // waits for its slowest workgroup, and their conflicts made the workgroups uneven.  Placed in pairs they cost
    // half, and the two ways take the same time, 0.68 of the LDS peak at N = 1e7, K = 1e4; a launch per round moves
    // less memory.)
    constexpr int64_t C = (THREADS / 2) * (int64_t)R;
    const int64_t nwg = (n_alloc + C - 1) / C;
    const int64_t per = rounds_per_launch > 0 ? (int64_t)rounds_per_launch * cu_count() : nwg;
    for (int64_t w0 = 0; w0 < nwg; w0 += per) {
        const int64_t cnt = nwg - w0 < per ? nwg - w0 : per;
        hipLaunchKernelGGL((assign_scan8q_kernel<R, THREADS, DEPTH>), dim3((unsigned)cnt), dim3(THREADS), 0, st, n_alloc - w0 * C,
                           gc8 + w0 * C, img, ntiles, assign, dist, ro);
        ++t_scan_kernels;
    }
}

void launch_scan_grouped8_q(int variant, const uint4* gc8, int64_t n_alloc, const float4* img, int ntiles,
                            int32_t* assign, float* dist, hipStream_t st, RankOut ro, int rounds_per_launch)
{
    int R = 0;
    switch (variant) {
        case 81: R = 24; break;
        case 82: R = 22; break;
        case 83: R = 20; break;
        case 84: R = 16; break;
        default: R = scan8q_codes_per_slot(n_alloc, nullptr); break;
    }
    switch (R) {
        case 16: launch_scan8q_rounds<16>(gc8, n_alloc, img, ntiles, assign, dist, st, ro, rounds_per_launch); break;
        case 20: launch_scan8q_rounds<20>(gc8, n_alloc, img, ntiles, assign, dist, st, ro, rounds_per_launch); break;
        case 22: launch_scan8q_rounds<22>(gc8, n_alloc, img, ntiles, assign, dist, st, ro, rounds_per_launch); break;
        default: launch_scan8q_rounds<24, 512, 2>(gc8, n_alloc, img, ntiles, assign, dist, st, ro, rounds_per_launch); break;
    }
}

// the same for 64-bit codes: zero the class counters, count, plan, scatter
pqkm_status regroup_codes8(const uint8_t* codes, int64_t cnt, uint4* gc8, GroupPlan8* plan, hipStream_t st,
                           bool blocks_of_16 = false)
{
    const int64_t na = group_alloc(cnt);
    if (blocks_of_16)
        hipLaunchKernelGGL(code8_group_clear_kernel, dim3(1024), dim3(256), 0, st, gc8, na);
    hipLaunchKernelGGL(zero_u32_kernel, dim3(64), dim3(256), 0, st, plan->count, (int64_t)GROUP8_CLASSES);
    unsigned g = (unsigned)((cnt + 1023) / 1024 < 4096 ? (cnt + 1023) / 1024 : 4096);
    if (g < 1) g = 1;
    hipLaunchKernelGGL(code8_class_count_kernel, dim3(g), dim3(256), 0, st, codes, cnt, plan);
    hipLaunchKernelGGL(code8_group_plan_kernel, dim3(1), dim3(1024), 0, st, plan);
    hipLaunchKernelGGL(code8_group_scatter_kernel, dim3(g), dim3(256), 0, st, codes, cnt, plan, gc8, na,
                       blocks_of_16 ? 1 : 0);
    return launched();
}

// regroup `cnt` codes into gco: three launches on the stream
pqkm_status regroup_codes(const uint8_t* codes, int64_t cnt, uint2* gco, GroupPlan* plan, hipStream_t st,
                          bool blocks_of_16 = false)
{
    const int64_t na = group_alloc(cnt);
    if (blocks_of_16)
        hipLaunchKernelGGL(code_group_clear_kernel, dim3(1024), dim3(256), 0, st, gco, na);
    int64_t g = (cnt + 4095) / 4096;
    if (g > GROUP_MAX_WGS) g = GROUP_MAX_WGS;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(code_class_count_kernel, dim3((unsigned)g), dim3(GROUP_THREADS), 0, st, codes, cnt, plan);
    hipLaunchKernelGGL(code_group_plan_kernel, dim3(1), dim3(1024), 0, st, plan, (int)g);
    hipLaunchKernelGGL(code_group_scatter_kernel, dim3((unsigned)g), dim3(GROUP_THREADS), 0, st, codes, cnt, plan, gco,
                       na, blocks_of_16 ? 1 : 0);
    return launched();
}

template <>
void launch_scan_M<4>(int variant, const uint8_t* codes, int64_t N, const float4* img, const float4* rows,
                      int ntiles, int32_t* assign, float* dist, hipStream_t st, const uint32_t*)
{
    switch (variant) {
        case 1: launch_scan<4, 16, 512, false>(codes, N, img, ntiles, assign, dist, st); break;
        case 3: launch_scan<4, 16, 512, true>(codes, N, img, ntiles, assign, dist, st); break;
        case 5: launch_scan<4, 8, 1024, false>(codes, N, img, ntiles, assign, dist, st); break;
        case 32: launch_scan4s<16, 768>(codes, N, img, ntiles, assign, dist, st); break;
        case 34: launch_scan4s<16, 1024>(codes, N, img, ntiles, assign, dist, st); break;
        case 36: launch_scan4s<16, 512>(codes, N, img, ntiles, assign, dist, st); break;
        case 37: launch_scan4s<8, 1024>(codes, N, img, ntiles, assign, dist, st); break;
        case 38: launch_scan4s<10, 1024>(codes, N, img, ntiles, assign, dist, st); break;
        case 39: launch_scan4s<12, 1024>(codes, N, img, ntiles, assign, dist, st); break;
        case 33: launch_scan4s<4, 512>(codes, N, img, ntiles, assign, dist, st); break;
        case 35: launch_scan4s<8, 512>(codes, N, img, ntiles, assign, dist, st); break;
        case 41: launch_scan4p<16, 1024, 1>(codes, N, nullptr, img, rows, ntiles, assign, dist, st); break;
        case 44: launch_scan4p<24, 512, 4>(codes, N, nullptr, img, rows, ntiles, assign, dist, st); break;
        case 46: launch_scan4p<28, 512, 3>(codes, N, nullptr, img, rows, ntiles, assign, dist, st); break;
        case 48: launch_scan4p<32, 512, 3>(codes, N, nullptr, img, rows, ntiles, assign, dist, st); break;
        default: launch_scan4s<16, 1024>(codes, N, img, ntiles, assign, dist, st); break;
    }
}
template <>
void launch_scan_M<8>(int variant, const uint8_t* codes, int64_t N, const float4* img, const float4* rows,
                      int ntiles, int32_t* assign, float* dist, hipStream_t st, const uint32_t* only_if)
{
    switch (variant) {
        case 1: launch_scan<8, 8, 512, false>(codes, N, img, ntiles, assign, dist, st); break;
        case 2: launch_scan_skew<8, 6, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 3: launch_scan_skew<8, 12, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 4: launch_scan_skew<8, 16, 512>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 5: launch_scan_skew<8, 24, 512>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 6: launch_scan_skew<8, 2, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 7: launch_scan_skew<8, 4, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 40: launch_scan8p<24, 512, 4>(codes, N, nullptr, img, ntiles, assign, dist, st); break;
        case 41: launch_scan8p<12, 1024, 2>(codes, N, nullptr, img, ntiles, assign, dist, st); break;
        default: launch_scan_skew<8, 8, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
    }
}
template <>
void launch_scan_M<16>(int variant, const uint8_t* codes, int64_t N, const float4* img, const float4* rows,
                       int ntiles, int32_t* assign, float* dist, hipStream_t st, const uint32_t* only_if)
{
    switch (variant) {
        case 1: launch_scan<16, 4, 512, false>(codes, N, img, ntiles, assign, dist, st); break;
        case 2: launch_scan_skew<16, 3, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 3: launch_scan_skew<16, 6, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 4: launch_scan_skew<16, 10, 512>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 6: launch_scan_skew<16, 2, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 7: launch_scan_skew<16, 1, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        default: launch_scan_skew<16, 4, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
    }
}
template <>
void launch_scan_M<32>(int variant, const uint8_t* codes, int64_t N, const float4* img, const float4* rows,
                       int ntiles, int32_t* assign, float* dist, hipStream_t st, const uint32_t* only_if)
{
    switch (variant) {
        case 1: launch_scan<32, 2, 512, false>(codes, N, img, ntiles, assign, dist, st); break;
        case 2: launch_scan_skew<32, 1, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 3: launch_scan_skew<32, 4, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 4: launch_scan_skew<32, 6, 512>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 5: launch_scan_skew<32, 8, 512>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        case 6: launch_scan_skew<32, 1, 512>(codes, N, img, ntiles, assign, dist, st, only_if); break;
        default: launch_scan_skew<32, 2, 1024>(codes, N, img, ntiles, assign, dist, st, only_if); break;
    }
}

// Which scan runs: for M = 4 with the default variant, the regrouped half-plane scan when there is enough work
// to pay for regrouping (a pass over the codes) and the subspace-skewed scan otherwise.
// M = 4, skewed scan of 2048 (37), 2560 (38), 3072 (39) or 4096 (34) codes per workgroup by the time of its rounds, from measured ones, us: one
// round 21 / 24.5 / 27.5 / 35 at K = 32, 45 / 50 / 56 / 76 at K = 200, 140 / 162 / 186 / 260 at K = 1000 (the last one spills registers).
struct SkewChoice { int variant; double us; };
SkewChoice choose_scan4s(int64_t N, int K)
{
    static const struct { int variant, codes; double round, tile; } shapes[] = {
        {37, 2048, 9.7, 3.85}, {38, 2560, 12.0, 4.43}, {39, 3072, 14.5, 5.1}, {34, 4096, 20.0, 7.25}};
    const int64_t ncu = cu_count();
    SkewChoice best{37, 1e300};
    for (const auto& s : shapes) {
        const double us = 8.0 + (double)(((N + s.codes - 1) / s.codes + ncu - 1) / ncu) * (s.round + s.tile * (double)((K + 31) / 32));
        if (us < best.us) best = SkewChoice{s.variant, us};
    }
    return best;
}

inline int effective_variant(int M, int variant, int64_t N, int K, const uint8_t* codes, const uint8_t* centers, bool alone)
{
    // the regrouped scans address the tile images through one 32-bit buffer offset: below 4 GB of images only
    const int TK = 128 / M;
    const bool img32 = (int64_t)((K + TK - 1) / TK) * TILE_BYTES < (int64_t)0xfff00000;
    const bool special = (variant >= 40 && variant <= 49) || (variant >= 70 && variant <= 79) ||
                         (M == 4 && variant >= 60 && variant <= 64) || (M == 8 && variant >= 60 && variant <= 63) || (M == 4 && variant >= 80 && variant <= 99) || (M == 8 && variant >= 80 && variant <= 84);
    if (M == 8) {
        const bool ok8 = img32 && ((uintptr_t)codes & 7) == 0;
        if (special && !ok8) return 0;
        // 65536 residue classes: regrouping pays once most classes hold a few dozen codes; then two lanes per code
        // (an LDS access holds two groups of four codes, so the left-over groups cost it more than the four-lane scan
        // 70, but a tile fill serves twice the codes: 0.63 against 0.60 of the LDS peak at N = 1e7, K = 1e4)
        // with enough centers for the lower-bound scan fewer codes pay for the regrouping as well (N = 1e6, K = 5000: 2.4 ms
        // with it against 2.6 ms of the skewed scan in a first iteration, 0.9 ms in later ones)
        if (variant == 0 && ok8 && ((K >= 256 && N >= ((int64_t)1 << 22)) ||
                                    (K >= filter8_min_k(0) && N >= ((int64_t)1 << 19) && (double)N * K >= 6e9 && ((uintptr_t)centers & 3) == 0)))
            return choose_scan8_large(N, K);
        if (variant == 0) {
            // skewed scan: while one round of workgroups covers the codes, the smallest shape that does so (measured
            // per round at K = 1000: 139, 172, 220, 263 us for 512, 1024, 1536, 2048 codes per workgroup)
            const int64_t ncu = cu_count();
            if (N <= ncu * 1536) return N <= ncu * 512 ? 6 : N <= ncu * 1024 ? 7 : 2;
            // then whichever of the two large ones takes less for its rounds: N = 524289, K = 100: 98 / 83 us, K = 400: 231 / 195
            auto rounds = [&](int64_t C) { return (double)((N + C * ncu - 1) / (C * ncu)); };
            return rounds(1536) * 0.84 < rounds(2048) ? 2 : 0;
        }
        return variant;
    }
    if ((M == 16 || M == 32) && variant == 0) {
        // the same for the wider codes (M = 16: 270, 343, 440, 524 us; M = 32: 640, 690, -, 1066 us); beyond one
        // round of those workgroups the sliding-window scan, whose workgroups take 2048 or 4096 codes
        const int64_t ncu = cu_count();
        if (M == 16) return N <= ncu * 512 ? 7 : N <= ncu * 1024 ? 6 : N <= ncu * 1536 ? 2 : 50;
        return N <= ncu * 512 ? 6 : N <= ncu * 1024 ? 2 : 50;
    }
    if (M == 4 && !img32 && special) return 34;
    if (M != 4 || variant != 0) return variant;
    // The skewed scan needs no regrouping pass and comes in shapes of 512 to 4096 codes per workgroup; a workgroup's
    // time grows with its codes (measured per round at K = 1000: 82, 107, 133, 254 us for 512, 1024, 2048, 4096),
    // so while one round of workgroups covers all codes the smallest shape that does so wins, also over the
    // regrouped scan (117 us and up per round plus the regrouping).  Beyond one round of 2048-code workgroups the
    // regrouped scan is faster where a fit uses the regrouped codes several times and K >= 128; else the skewed shape with the
    // fewest microseconds, and for one assignment by itself the faster of the two.
    const int64_t ncu = cu_count();
    if (N <= ncu * 512) return 33;
    if (N <= ncu * 1024) return 35;
    if (N <= ncu * 2048) return 37;
    const SkewChoice best = choose_scan4s(N, K);
    if (K < 128 || !img32) return best.variant;
    // regrouping and the rest 25 us and 40 ps per code, and the rounds of choose_scan4_large.  One assignment, regrouped / skewed, us: K = 200:
    // 87 / 51 at N = 655360, 146 / 109 at 1.57e6, 165 / 148 at 2e6; K = 500: 142 / 104 at 786432, 201 / 172 at 1.28e6, but 256 / 275 at 2e6; K =
    // 1000: 193 / 165 at 655360, 305 / 262 at 1048576, but 356 / 365 at 1.57e6.
    if (alone && K < filter4_min_k(0, N)) {
        double clocks;
        choose_scan4_large(N, &clocks);
        if (best.us < 0.97 * (25.0 + 4e-5 * (double)N + clocks * (double)((K + 31) / 32) / 2200.0)) return best.variant;
    }
    return 70;                            // regrouped half-plane scan, codes per lane-slot chosen per launch
}
inline bool variant_filter(int M, int variant)
{
    return (M == 4 && variant >= 60 && variant <= 64) || (M == 8 && variant >= 60 && variant <= 63);
}
inline bool variant_grouped(int M, int variant)
{
    return variant_filter(M, variant) || ((M == 4 || M == 8) && variant >= 70 && variant <= 79) || (M == 4 && variant >= 80 && variant <= 99) ||
           (M == 8 && variant >= 80 && variant <= 84);
}
inline bool variant_two_lane(int M, int variant)
{
    return variant_filter(M, variant) || (M == 4 && variant >= 80 && variant <= 99) ||
           (M == 8 && variant >= 80 && variant <= 84);
}
inline bool variant_table_tiles(int M, int variant) { return M == 4 && variant >= 90 && variant <= 99; }
inline bool variant_lds_loads(int M, int variant) { return M == 4 && variant >= 85 && variant <= 89; }
inline bool variant_sliding(int M, int variant) { return (M == 16 || M == 32) && variant >= 50 && variant <= 59; }

// Histogram with all clusters of G subspaces in a workgroup's LDS (G = 0: not taken): about one workgroup per compute unit,
// slices of at least 2048 codes, at most 64, whose partial arrays fit the room of the sorted path: of 16-bit counters (halves) where
// that leaves no more codes per slice than they count.
struct SubspaceHist { int G, S; bool halves; };
SubspaceHist subspace_hist(int64_t N, int M, int K, const Carve& c)
{
    SubspaceHist p{0, 1, false};
    // Every workgroup reads a word of every code of its slice, whatever M is, and leaves K G KB for the vote to add; the owner
    // path reads a byte per code and group, but a heavy cluster is the work of one of its workgroups.  Clusters of even / of uneven size (the cube of a
    // random number), whole update, owner : this, us: M = 4, K = 100: 28.5 : 31.4 / 39.8 : 31.2 at N = 4e5, 37.5 : 31.5 / 57.7 : 31.2 at 8e5, 89.7 : 40.0 / 184 :
    // 39.8 at 3.2e6; M = 8, K = 48: 49.8 : 34.8 / 100 : 34.9 at 8e5; K = 100: 66.7 : 50.4 / 151 : 50 at 1.6e6; M = 16, K = 48: 67 : 44 / 161 : 44 at 8e5; M = 32, K =
    // 20: 104 : 64 / 177 : 65 at 8e5.  32 clusters of four subspaces per workgroup are fewer workgroups: M = 4: 32.6 : 34.3 at 8e5, 47.0 : 39.6 at 1.6e6; M = 12: 33.3
    // : 36.5 at 1e6 where members share subcodes.  Taken where it does not cost even clusters more than a few per cent.  With fewer than 32 centers that was
    // so until the owner path formed its adds in line (M = 32, K = 28, 1.25e6: 73 : 111 / 280 : 111; M = 64, K = 16, 1.6e6: 117 : 149 / 378 : 147): kept for the
    // uneven ones.  From 32 centers on, where the owner path's figures above are of before too, none of 800 random sizes loses more than 3 % by the rule.
    if (N > (int64_t)0xffffffff || (int64_t)K * L > SUBSPACE_HIST_WORDS) return p;
    const int64_t least = K == 32 ? (M == 4 ? 1200000 : 1500000) : 1000000;
    if (N < least || !(K >= 32 ? M >= 4 && M <= 16 : M >= 16)) return p;
    p.G = 1;
    while (p.G < 4 && p.G * 2 <= M && (int64_t)K * L * p.G * 2 <= SUBSPACE_HIST_WORDS) p.G *= 2;
    const int64_t groups = (M + p.G - 1) / p.G;
    auto slices = [&](size_t part_bytes) {
        const int64_t room = (int64_t)(c.seg_off - c.sidx_off) / (int64_t)align256(part_bytes);
        const int64_t most[] = {room, cu_count() / groups, N / 2048, 64};
        int64_t S = most[0];
        for (int64_t x : most) S = x < S ? x : S;
        // Workgroup (g, s) runs on die s mod 8 where S is a multiple of eight, so that the groups of a slice share one L2's copy of its codes: M = 48, K = 7,
        // 2.5e6 codes: 93 us with 16 slices, 174 with 21.
        if (groups > 1 && S > 8) S &= ~(int64_t)7;
        return (int)(S < 1 ? 1 : S);
    };
    p.S = slices((size_t)K * M * L * sizeof(uint16_t));
    p.halves = p.S > 1 && ((N + p.S - 1) / p.S + 1023) / 1024 * 1024 <= SUBSPACE_HALF_CODES;
    if (!p.halves) p.S = slices((size_t)K * M * L * sizeof(uint32_t));
    // With fewer slices (no room for their arrays) the chip is half idle, owner : this: M = 8, K = 128: 41.5 : 60.6 with 6 at 8e5, 62.2 : 61.3 with 12 at 1.6e6; M =
    // 16, K = 64: 55.3 : 73.6 with 6; with 12, where all codes are alike, 123 : 136.
    if (K >= 32 && p.S < 16) p.G = 0;
    return p;
}

// How the update counts its histograms: from the records of the fused iteration (`linked`), per cluster group, per group of
// subspaces, from the indices sorted by cluster, or by global atomics.
enum HistPath { HIST_RECORDS, HIST_OWNER, HIST_SUBSPACE, HIST_SORTED, HIST_ATOMIC };
HistPath hist_path(int64_t N, int M, int K, const Carve& c, int force, bool linked, bool keys)
{
    const HistPlan hp = hist_plan(N, M, K);
    if (owner_histogram(hp, force)) {
        if (linked) return HIST_RECORDS;
        if (force == 0 && subspace_hist(N, M, K, c).G > 0) return HIST_SUBSPACE;
        if (force != 0 || !sorted_histogram_pays(hp, N, M, K, keys)) return HIST_OWNER;
    }
    return force != 1 && N <= (int64_t)0xffffffff && N > 0 ? HIST_SORTED : HIST_ATOMIC;
}

// The fused iteration's hand-over from the scan to the histogram: filled in by the caller (wanted, KT, ngroups),
// completed by the assignment (produced, nwg) when the scan that ran could file its codes by cluster group.
struct BucketLink {
    bool wanted = false, produced = false;
    int KT = 0, ngroups = 0, nwg = 0;
    // the other hand-over (sorted-path sizes): every code's rank inside its cluster, counted by the scan's epilogue
    bool rank_wanted = false, ranked = false;
};

// M = 16, 32: is the lower-bound scan tried before the sliding-window scan?  (Neither then leaves ranks for the histogram:
// those of a scan that gave up could not be taken back.  The update's own counting and block-wise scatter take as long as
// placing the codes by rank.)
constexpr int FILTER_WIDE_PAIRS_MIN_K = 500;
// Fewest centers, by iteration, as for M = 4.  Measured at N = 1e6 against the sliding-window scan, ms per iteration, M = 32:
// first 5.1 / 3.8 at K = 2000, 12.4 / 16.4 at 10000; second and third 5.0 / 3.95 and 12.1 / 17.3; later 3.4 / 3.95 and
// 9.5 / 17.3.  M = 16, K = 3000: 2.9 / 2.9, 2.3 / 3.0, 1.7 / 3.0.
inline int wide_min_k(int M, int iteration)
{
    return M == 32 ? (iteration == 0 ? 5000 : iteration < 3 ? 4000 : 1500) : (iteration == 0 ? 3500 : iteration < 3 ? 1800 : 900);
}
inline bool wide_filter(int M, int asked, int variant, int64_t N, int K, const uint8_t* centers, int iteration)
{
    if ((M != 16 && M != 32) || !variant_sliding(M, variant)) return false;
    if (((uintptr_t)centers & 3) != 0 || ((int64_t)K + 63) / 64 * (M * 16384) >= (int64_t)0xfff00000) return false;
    if (K <= 64) return false;                           // the byte tables take 16 KB + 64 KB M of the histograms' room, M KB per center
    if (asked == 59) return true;                        // forced
    return asked == 0 && K >= wide_min_k(M, iteration);
}

template <int M>
void launch_filter_wide(const uint8_t* codes, int64_t N, uint32_t* S, FilterWideIn f, int32_t* assign, float* dist,
                        hipStream_t st)
{
    const int ncu = cu_count();
    constexpr int64_t C = 1024;                          // more codes per workgroup do not fit the registers
    const int64_t nwg = (N + C - 1) / C;
    f.S = S;
    f.n_alloc = nwg * C;
    f.spent = S + (size_t)(M / 4) * f.n_alloc;           // the room has a word per code more than the rotated words take
    f.codes = codes;
    hipLaunchKernelGGL((code_rotate_kernel<M>), dim3((unsigned)((f.n_alloc + 255) / 256)), dim3(256), 0, st, codes, N, S, f.n_alloc, f.only_if);
    // tiles per launch: all of them while there is one round of workgroups
    const int step = nwg <= ncu ? f.ntiles : (4 << 20) / (M * (int)FILTER_PLANE);
    for (int t0 = 0; t0 < f.ntiles; t0 += step)
        for (int64_t w0 = 0; w0 < nwg; w0 += ncu) {      // a round of workgroups per launch: they start in step
            const unsigned cnt = (unsigned)(nwg - w0 < ncu ? nwg - w0 : ncu);
            f.t_begin = t0;
            f.t_end = f.ntiles - t0 < step ? f.ntiles : t0 + step;
            hipLaunchKernelGGL((assign_filter_wide_kernel<M, 2, 1024>), dim3(cnt), dim3(1024), 0, st, N, f, assign, dist, w0);
            ++t_scan_kernels;
        }
}

// What the iterations of one call (same codes, tables and options) leave in the workspace for the next one.  Successive
// iterations may run different scans, in stretches of different length, so nothing follows from the iteration's number alone.
struct Carried {
    int iteration = 0;        // of the assignment step about to run; > 0: assign[] holds the result of the one before
    int lanes = 0;            // a regrouped copy of ALL codes, placed for slots of this many lanes (0: there is none)
    bool stats = false;       // the lower-bound scan's statistics of the tables
    bool keys = false;        // its keys by position in that copy, and the copy of the centers that they belong to
    bool alone = false;       // one assignment by itself, not an iteration of a fit
    bool dot = false;         // the points of the scan on the matrix cores, or that it is not for these tables
};

// Is the scan on the matrix cores tried first, and for how many dimensions?  Whole calls take up to 4e12 center-code pairs per
// second at 128 dimensions (M = 8, N = 1e6, K = 4000) and half of that at 256, behind 10 to 27 us for the points, once per call, and
// 8 for the centers' fragments, and a block of codes costs 10 to 13 us beside its centers; tables it is not for cost 10 us (M = 8: 14,
// 20 where they take few values).  The distances, where they are asked for, are M table entries per code from the L2 (18 us at M =
// 16, N = 250007).  Whole calls, plain scans / this, us, where this is taken and where it is not.
// M = 8, with distances, 128 dimensions: 150 / 69 at N = 1e5, K = 1000; 106 / 76 at 2e5, 500; 574 / 342 at 1e6, 1000; but 84 / 81 at 3e5,
// 300; 215 / 208 at 2e6, 100.  256 dimensions: 148 / 113 at 1e5, 1000; 190 / 153 at 1.8e5, 1000; 541 / 483 at 4e5, 2000; but 103 /
// 123 at 2e5, 500; 184 / 186 at 2.6e5, 1000; 305 / 320 at 5e5, 1000; 562 / 582 at 1e6, 1000: by the rounds of both.
// M = 16, with distances, 128: 51 / 44 at 1e5, 130; 127 / 39 at 25100, 400; 187 / 159 at 1e6, 100; 205 / 177 at 1.2e6, 72; but 57 / 58
// at 2e5, 100; 139 / 142 at 1e6, 64.  256: 66 / 46 at 6e4, 200; 131 / 103 at 2e5, 300; but 91 / 94 at 2e5, 200.  Without distances, 128:
// 41 / 39 at 1.5e5, 64; 103 / 83 at 1e6, 20; 74 / 66 at 6e5, 25; but 42 / 45 at 3e5, 32.  256: 99 / 88 at 3.5e5, 103; 51 / 50 at 1e5,
// 130; 169 / 160 at 1e6, 90; but 137 / 145 at 1e6, 64.
// M = 32, with, 128: 90 / 60 at 1e5, 100; 150 / 119 at 3e5, 80; 265 / 244 at 1e6, 64; but 83 / 84 at 2e5, 64.  256: 91 / 72 at 1e5, 100; 75
// / 69 at 1e5, 80; 376 / 346 at 1e6, 100; but 305 / 324 at 1e6, 80.  Without, 128: 100 / 65 at 5e5, 20; 70 / 49 at 2.5e5, 40.  256: 78 / 55 at 1.2e5, 80; 224 /
// 165 at 1e6, 40; 96 / 73 at 3e5, 31; 199 / 152 at 6.7e5, 54 (but 269 / 441 at 1e6, 64, left, where no code lies near a center).
// This is for sizes with an LDS-tiled scan behind it; below gather_max_codes dot_before_rows decides.  The
// sizes at which M = 8 regroups its codes are left to the lower-bound scan (up to 8.7e12 pairs per second in later iterations, 2e12 in
// a first one), and all of M = 4 to its scans.
int dot_scan_dims(int M, const Options& opt, int64_t N, int K, bool dist, const uint8_t* centers, const Carve& c)
{
    if (c.dot_off == 0 || ((uintptr_t)centers & 3) != 0 || (int64_t)K > ((int64_t)1 << 22)) return 0;
    if (opt.scan_variant == 20) return 256;              // forced
    if (opt.scan_variant != 0) return 0;
    const double pairs = (double)N * K;
    if (M == 8) {
        if (pairs < 9e7 || K < 500) return 0;
        // 256 dimensions, us: 45 and rounds of 256 codes per compute unit, against the rounds of the skewed scan (effective_variant)
        const int64_t ncu = cu_count();
        const double rounds = (double)((N + 256 * ncu - 1) / (256 * ncu)) * (13.0 + 0.0205 * K);
        const double plain = 0.001 * K * (N <= ncu * 512 ? 139.0 : N <= ncu * 1024 ? 172.0 : N <= ncu * 1536 ? 220.0 : 263.0 * (double)((N + 2048 * ncu - 1) / (2048 * ncu)));
        return 45.0 + rounds < 0.95 * (12.0 + plain) ? 256 : 128;
    }
    if (pairs < 9e6 || (M == 16 && N < 25000)) return 0;
    if (M == 16 && dist) return K < (pairs < 5e7 ? 110 : 70) ? 0 : K >= (N < 150000 ? 180 : 300) ? 256 : 128;
    if (M == 16) return K < (pairs < 1.3e7 ? 64 : 17) ? 0 : K >= 80 ? 256 : 128;
    if (dist) return K < (pairs < 1.6e7 ? 80 : 64) ? 0 : K >= (N < 400000 ? 80 : 100) ? 256 : 128;
    return K < 16 ? 0 : 256;
}

template <int M, bool MARKS>
void launch_dot(const uint8_t* codes, int64_t N, const uint8_t* centers, int K, const float* tables, int32_t* assign, float* dist,
                const Carve& c, char* ws, const Carried& carried, const Options& opt, int most_dims, hipStream_t st)
{
    const DotCarve d = dot_carve(M, K);
    char* room = ws + c.img_off;
    DotState* state = reinterpret_cast<DotState*>(ws + c.dot_off);
    DotStat* stat = reinterpret_cast<DotStat*>(room + d.stat_off);
    DotCheck* check = reinterpret_cast<DotCheck*>(room + d.check_off);
    _Float16* emb = reinterpret_cast<_Float16*>(room + d.emb_off);
    float* lost = reinterpret_cast<float*>(room + d.lost_off);
    if (!carried.dot)
        hipLaunchKernelGGL((dot_points_kernel<M>), dim3(M * DOT_PARTS), dim3(256), 0, st, tables, stat, check, emb, lost, state, most_dims);
    hipLaunchKernelGGL((dot_centers_kernel<M>), dim3((unsigned)((K + DOT_TILE - 1) / DOT_TILE)), dim3(256), 0, st, centers, K, stat,
                       check, emb, lost, state, room + d.img_off, carried.iteration, !carried.dot);
    EventPair ev{};
    const bool prof = (opt.profile & 1) && log_begin(g_scan_log, st, &ev);
    const DotIn in{codes, centers, tables, stat, emb, lost, room + d.img_off, state, N, K, carried.iteration};
    const int64_t ncu = cu_count();
    // one or two columns of codes per wave, by the time of the rounds: about 20 tiles' worth for what a round costs beside its tiles
    auto cost = [&](int64_t ct) { return (double)(((N + 256 * ct - 1) / (256 * ct) + ncu - 1) / ncu) * ((double)K / DOT_TILE * (double)ct + 20.0); };
    const int ct = cost(2) <= cost(1) ? 2 : 1;
    const int64_t blocks = (N + 256 * ct - 1) / (256 * ct);
    const dim3 grid((unsigned)(blocks < ncu ? blocks : ncu));
    if (ct == 2) hipLaunchKernelGGL((assign_dot_kernel<M, 2, MARKS>), grid, dim3(512), 0, st, in, assign, dist);
    else hipLaunchKernelGGL((assign_dot_kernel<M, 1, MARKS>), grid, dim3(512), 0, st, in, assign, dist);
    if (prof) {
        hipEventRecord(ev.b, st);
        std::lock_guard<std::mutex> lk(g_mu);
        ++g_scan_log.kernels;
    }
}

struct ScanPlan {
    int variant;
    bool filter, wide, grouped, sliding;
    int dot;                  // dimensions up to which the scan on the matrix cores is tried first; the above is for what it leaves
    int lanes;                // lanes per slot that the regrouped copy is placed for (grouped)
    int64_t per_launch;       // codes per stretch
    bool reuse;               // the regrouped copy is there already
    int seeded;               // filter: FilterIn::seeded
    Carried leaves;           // for the next iteration
};

// Which scan an assignment step runs, in which stretches, and what it can take over from the iteration before: host
// arithmetic, without a look at the device's memory.
ScanPlan scan_plan(int M, const Options& opt, int64_t N, int K, const uint8_t* codes, const uint8_t* centers, bool files_records,
                   bool dist, const Carve& c, const Carried& had)
{
    ScanPlan p{};
    const int iteration = had.iteration;
    const int asked = opt.scan_variant == 20 ? 0 : opt.scan_variant;      // 20: the scan on the matrix cores in front of the default ones
    int variant = effective_variant(M, asked, N, K, codes, centers, had.alone);
    // No records to file for the histogram: the four-lane scan or the scan with two-lane slots whose tiles are loaded
    // straight into LDS, half a tile ahead, in the shape that the rounds favour
    // Records to file (the fused iteration at owner-path sizes): the same scan in its 4096-code shape, which files
    // them as the four-lane scan does.
    // The lower-bound scan addresses its byte tiles through one 32-bit buffer offset and reads centers as words.
    const bool filter_ok = (M == 4 || (M == 8 && K > 16 && c.side_off > 0)) && ((uintptr_t)centers & 3) == 0 && ((int64_t)K + 63) / 64 * (M * 16384) < (int64_t)0xfff00000;
    if (M == 4 && variant == 70 && asked == 0)
        variant = filter_ok && K >= filter4_min_k(iteration, N) ? (files_records ? 63 : 60)
                  : files_records ? 89 : choose_scan4_large(N);
    else if (variant_filter(M, variant) && !filter_ok)
        variant = M == 4 ? 85 : 80;
    if (M == 8 && asked == 0 && variant_grouped(8, variant) && filter_ok && K >= filter8_min_k(iteration)) variant = 60;
    if (M == 4 && variant == 65) variant = files_records ? 89 : choose_scan4_large(N);      // the best of the plain scans
    p.variant = variant;
    p.filter = variant_filter(M, variant);
    p.grouped = variant_grouped(M, variant);
    p.sliding = variant_sliding(M, variant);
    // M = 16, 32: the lower-bound scan of every stretch in front of the sliding-window scan, which runs where it gave up
    p.wide = p.sliding && wide_filter(M, asked, variant, N, K, centers, iteration);
    p.dot = p.grouped ? 0 : dot_scan_dims(M, opt, N, K, dist, centers, c);
    p.lanes = !p.grouped ? 0 : variant_two_lane(M, variant) ? 2 : 4;
    int64_t per_launch = opt.launch_codes;
    // a little below the limit: with its padding a launch of exactly 2^26 codes needs one workgroup more than
    // 64 full rounds of 4096-code workgroups, and that workgroup would run a round of its own
    if ((p.grouped || p.sliding) && per_launch > GROUP_CHUNK_MAX - 16384) per_launch = GROUP_CHUNK_MAX - 16384;
    if (p.filter) {
        const int64_t round = (int64_t)cu_count() *
                              (M == 4 ? 512 * filter4_codes_per_slot(variant, group_alloc(N)) : 256 * filter8_codes_per_slot(variant, group_alloc(N)));
        if (per_launch >= round) per_launch = per_launch / round * round - 32;
    }
    if (variant_lds_loads(M, variant)) {
        // whole rounds of these large workgroups per stretch (the regrouped copy pads a stretch by less than 32 codes)
        const int64_t round = (int64_t)cu_count() * scan4h_codes_per_workgroup(variant);
        if (per_launch >= round) per_launch = per_launch / round * round - 32;
    }
    p.per_launch = per_launch;
    const bool one = N <= per_launch;
    p.reuse = p.grouped && one && had.lanes == p.lanes;
    // A first iteration starts from the centers that share a pair of subcodes with the code, a later one from the center of
    // the one before: by code position where the keys are there, else through assign[].
    if (p.filter) p.seeded = iteration == 0 ? (K >= FILTER_PAIRS_MIN_K ? 3 : 0) : had.keys && p.reuse ? 2 : 1;
    // the keys stay unless the update uses their room (that of the sorted path, and of the arrays of HIST_SUBSPACE); of the scans with
    // keys only M = 4's 63 files records
    const HistPath path = hist_path(N, M, K, c, opt.hist_kernel, files_records && variant == 63 && one, scans_keep_keys(M));
    const bool keys_survive = c.state_off != c.sidx_off || path == HIST_RECORDS || path == HIST_OWNER;
    p.leaves.iteration = iteration + 1;
    p.leaves.lanes = one ? p.lanes : 0;
    p.leaves.stats = p.filter;
    p.leaves.keys = p.filter && one && keys_survive;
    p.leaves.dot = p.dot > 0;
    return p;
}

template <int M>
pqkm_status assign_tiled(const uint8_t* codes, int64_t N, const uint8_t* centers, int K, const float* tables,
                         int32_t* assign, float* dist, float* img, const Options& opt, const Carve& c, char* ws,
                         Carried& carried, hipStream_t st, BucketLink* link = nullptr)
{
    constexpr int TK = 128 / M;
    int64_t ntiles = ((int64_t)K + TK - 1) / TK;
    int64_t total = ntiles * (int64_t)(TILE_BYTES / 4);
    const int iteration = carried.iteration;
    const bool files_records = M == 4 && link && link->wanted && N <= GROUP_CHUNK_MAX - 16384 && c.bseg_off != c.pool_off;
    const ScanPlan plan_of = scan_plan(M, opt, N, K, codes, centers, files_records, dist != nullptr, c, carried);
    const int variant = plan_of.variant;
    const bool filter = plan_of.filter, wide = plan_of.wide, grouped = plan_of.grouped, sliding = plan_of.sliding;
    const int64_t per_launch = plan_of.per_launch;
    const int layout = variant_layout(M, variant);
    // not NULL: a word that says whether the scans below have anything to do
    const uint32_t* left = nullptr;
    if constexpr (M != 4) {
        if (plan_of.dot) {
            launch_dot<M, false>(codes, N, centers, K, tables, assign, dist, c, ws, carried, opt, plan_of.dot, st);
            if (launched() != PQKM_OK) return PQKM_ERR_DEVICE;
            left = &reinterpret_cast<const DotState*>(ws + c.dot_off)->left;
        }
    }
    // images that may not be needed are built by few blocks
    auto blocks_of = [&](int64_t elements) {
        const int64_t b = (elements + 255) / 256;
        return (unsigned)(left && b > 2048 ? 2048 : b);
    };
    // The statistics of the M = 16, 32 lower-bound scan live in the histograms' room while the assignment runs, its byte tiles
    // and pair tables in that of the images, which are only built after a scan has given up.
    FilterStat* const wstat = reinterpret_cast<FilterStat*>(ws + c.hist_off);
    FilterScale* const wscale = reinterpret_cast<FilterScale*>(ws + c.hist_off + 8192);
    uint32_t* const gave_up = reinterpret_cast<uint32_t*>(ws + c.hist_off + 8448);
    uint32_t* const wbytes = reinterpret_cast<uint32_t*>(ws + c.hist_off + 16384);
    // M = 4, 8: byte tiles in the room of the images, which are built there only for codes that the scan left; the pair tables in
    // that of the row-ordered images (M = 4) or behind the byte tiles, which take a quarter of the images' room (M = 8: at most
    // 1 MB).  What lasts until the next iteration has a room of its own: statistics, the scale, two copies of the centers (this
    // iteration's and the one before).
    char* const side = M == 4 ? ws + c.tabt_off : ws + c.side_off;
    const int nt64 = (K + FILTER_TK - 1) / FILTER_TK;
    FilterIn fin{};
    uint32_t* pairs = nullptr;
    uint8_t* this_copy = nullptr;
    if (filter) {
        static_assert(M * FILTER_PARTS * sizeof(FilterStat) <= 4096, "statistics");
        uint8_t* copies = M == 4 ? reinterpret_cast<uint8_t*>(ws + c.rowoff_off) : reinterpret_cast<uint8_t*>(side + 4096 + 512);
        const size_t copy_stride = align256((size_t)K * M);
        this_copy = copies + (iteration & 1) * copy_stride;
        pairs = reinterpret_cast<uint32_t*>(M == 4 ? ws + c.rows_off : ws + c.img_off + align256((size_t)nt64 * M * FILTER_PLANE));
        fin = FilterIn{reinterpret_cast<const uint4*>(img), tables, centers, reinterpret_cast<FilterScale*>(side + 4096),
                       reinterpret_cast<unsigned long long*>(ws + c.state_off), K, nt64, copies + ((iteration & 1) ^ 1) * copy_stride,
                       pairs, plan_of.seeded, reinterpret_cast<uint32_t*>(side + 4096 + 256), 0};
    } else if (sliding) {
        // tiles of 16 centers, plane-ordered: img[tile][m][x][16]
        ntiles = ((int64_t)K + 15) / 16;
        total = ntiles * (int64_t)16 * M * L;
        if (!wide) hipLaunchKernelGGL((tile_image_kernel<M, 0, 16>), dim3(blocks_of(total)), dim3(256), 0, st,
                           centers, K, tables, img, total, (float*)nullptr, left);
    } else if (layout == 2 && M == 4)
        hipLaunchKernelGGL((tile_image_kernel<4, 2>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                           centers, K, tables, img, total, reinterpret_cast<float*>(ws + c.rows_off));
    else if (layout == 1)
        hipLaunchKernelGGL((tile_image_kernel<M, 1>), dim3(blocks_of(total)), dim3(256), 0, st,
                           centers, K, tables, img, total, (float*)nullptr, left);
    else
        hipLaunchKernelGGL((tile_image_kernel<M, 0>), dim3(blocks_of(total)), dim3(256), 0, st,
                           centers, K, tables, img, total, (float*)nullptr, left);
    if (launched() != PQKM_OK) return PQKM_ERR_DEVICE;
    const float4* rows = reinterpret_cast<const float4*>(ws + c.rows_off);
    uint2* gco = reinterpret_cast<uint2*>(ws + c.gco_off);
    GroupPlan* plan = reinterpret_cast<GroupPlan*>(ws + c.plan_off);
    uint4* gc8 = reinterpret_cast<uint4*>(ws + c.gc8_off);
    GroupPlan8* plan8 = reinterpret_cast<GroupPlan8*>(ws + c.plan8_off);
    // tiles built in the kernel from the transposed tables: the tables and the centers' row offsets, once per call
    TileSource tsrc{};
    if (variant_table_tiles(M, variant)) {
        float* tabT = reinterpret_cast<float*>(ws + c.tabt_off);
        uint32_t* rowoff = reinterpret_cast<uint32_t*>(ws + c.rowoff_off);
        hipLaunchKernelGGL(transpose_tables_kernel, dim3(L, (unsigned)M + 1), dim3(256), 0, st, tables, M, tabT);
        const int64_t nro = ntiles * 128;
        hipLaunchKernelGGL(tile_rows4_kernel, dim3((unsigned)((nro + 255) / 256)), dim3(256), 0, st, centers, K, rowoff, nro);
        tsrc.tabT = tabT;
        tsrc.rowoff = rowoff;
        tsrc.tab_bytes = (uint32_t)(((size_t)M * L + 1) * L * sizeof(float));
    }
    // ranks for the sorted-path histogram: from the scans that finish their codes one per lane (the regrouped scans
    // and the sliding-window scan), unless this iteration already hands records over by cluster group
    RankOut ro{};
    if (link && link->rank_wanted && (grouped || sliding) && !wide && !left && !(M == 4 && link->wanted && (variant == 70 || filter) && N <= per_launch)) {
        ro.count = reinterpret_cast<uint32_t*>(ws + c.seg_off);
        ro.rank = reinterpret_cast<uint32_t*>(ws + c.rank_off);
        unsigned zb = (unsigned)((K + 255) / 256 < 1024 ? (K + 255) / 256 : 1024);
        hipLaunchKernelGGL(zero_u32_kernel, dim3(zb), dim3(256), 0, st, ro.count, (int64_t)K);
        link->ranked = true;
    }
    // images that are built only for codes that a lower-bound scan left: a launch of 1024 blocks that stride costs less than one of 8192
    // where it ends at once, and calls that do give up take as long (0.98 to 1.01 times, M = 4 to 32, K = 1800 to 20000)
    const unsigned left_blocks = (unsigned)((total + 255) / 256 < 1024 ? (total + 255) / 256 : 1024);
    for (int64_t n0 = 0; n0 < N; n0 += per_launch) {
        int64_t cnt = N - n0 < per_launch ? N - n0 : per_launch;
        const RankOut rl{ro.count, ro.count ? ro.rank + n0 : nullptr};
        if (filter) {
            // for every stretch anew: the plain scan of the one before may have needed the room
            FilterStat* stat = reinterpret_cast<FilterStat*>(side);
            if (n0 == 0 && !carried.stats)
                hipLaunchKernelGGL(filter_stats_kernel, dim3(M * FILTER_PARTS), dim3(1024), 0, st, tables, stat);
            if constexpr (M < 16)
                hipLaunchKernelGGL((filter_image_kernel<M>), dim3((unsigned)(nt64 * M * 4)), dim3(256), 0, st, centers, K, tables, stat,
                                   reinterpret_cast<uint4*>(img), this_copy, reinterpret_cast<FilterScale*>(side + 4096), fin.gave_up);
            if (plan_of.seeded == 3) {
                hipLaunchKernelGGL(fill_i32_kernel, dim3(256), dim3(256), 0, st, reinterpret_cast<int32_t*>(pairs), (int64_t)(M / 2) * 65536, (int32_t)-1);
                hipLaunchKernelGGL((filter_pairs_kernel<M>), dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, centers, K, pairs);
            }
        }
        if (grouped && !plan_of.reuse) {
            const pqkm_status rs = (M == 8) ? regroup_codes8(codes + n0 * M, cnt, gc8, plan8, st, plan_of.lanes == 2)
                                            : regroup_codes(codes + n0 * M, cnt, gco, plan, st, plan_of.lanes == 2);
            if (rs != PQKM_OK) return PQKM_ERR_DEVICE;
        }
        EventPair ev{};
        const bool prof = (opt.profile & 1) && log_begin(g_scan_log, st, &ev);
        t_scan_kernels = 0;
        if (sliding) {
            if constexpr (M == 16 || M == 32) {
                if (wide) {
                    const bool pairs = iteration == 0 && K >= FILTER_WIDE_PAIRS_MIN_K;
                    const int nt = (K + FILTER_TK - 1) / FILTER_TK;
                    uint32_t* pair_tab = reinterpret_cast<uint32_t*>(img) + (size_t)nt * M * (FILTER_PLANE / 4);
                    // a stretch before this one may have given up and built the plain images in their place
                    if (n0 == 0) hipLaunchKernelGGL(filter_stats_kernel, dim3(M * FILTER_PARTS), dim3(1024), 0, st, tables, wstat, left);
                    hipLaunchKernelGGL((filter_bytes_kernel<M>), dim3(M * 16), dim3(256), 0, st, tables, wstat, wbytes, wscale, gave_up, left);
                    hipLaunchKernelGGL((filter_wide_image_kernel<M>), dim3((unsigned)(nt * M * 4)), dim3(256), 0, st, centers, K,
                                       reinterpret_cast<const uint4*>(wbytes), reinterpret_cast<uint4*>(img), left);
                    if (pairs) {
                        hipLaunchKernelGGL(fill_i32_kernel, dim3(256), dim3(256), 0, st, reinterpret_cast<int32_t*>(pair_tab),
                                           (int64_t)FILTER_WIDE_PAIRS * 65536, (int32_t)-1, left);
                        hipLaunchKernelGGL((filter_pairs_kernel<M, FILTER_WIDE_PAIRS>), dim3((unsigned)((K + 255) / 256)), dim3(256),
                                           0, st, centers, K, pair_tab, left);
                    }
                    launch_filter_wide<M>(codes + n0 * M, cnt, reinterpret_cast<uint32_t*>(ws + c.skew_off),
                                          FilterWideIn{reinterpret_cast<const uint4*>(img), nullptr, 0, nullptr, centers, tables, wscale,
                                                       reinterpret_cast<unsigned long long*>(ws + c.state_off),
                                                       pairs ? pair_tab : nullptr, gave_up, nullptr, K, 0, nt, nt, iteration > 0 ? 1 : 0,
                                                       left},
                                          assign + n0, dist ? dist + n0 : nullptr, st);
                    // what follows ends at once unless that scan gave up
                    hipLaunchKernelGGL((tile_image_kernel<M, 0, 16>), dim3(left_blocks), dim3(256), 0, st,
                                       centers, K, tables, img, total, (float*)nullptr, (const uint32_t*)gave_up);
                }
                if (launch_scan_sw<M>(variant, codes + n0 * M, cnt, reinterpret_cast<uint32_t*>(ws + c.skew_off),
                                      reinterpret_cast<const float4*>(img), (int)ntiles, assign + n0,
                                      dist ? dist + n0 : nullptr, st, rl, wide ? 0 : opt.rounds_per_launch,
                                      wide ? gave_up : left) != PQKM_OK)
                    return PQKM_ERR_DEVICE;
            }
        } else if (filter && M == 8) {
            if constexpr (M == 8) {
                launch_filter8(variant, gc8, group_alloc(cnt), fin, assign + n0, dist ? dist + n0 : nullptr, st, rl,
                               opt.rounds_per_launch);
                hipLaunchKernelGGL((tile_image_kernel<8, 0>), dim3(left_blocks), dim3(256), 0, st, centers, K, tables, img, total,
                                   (float*)nullptr, (const uint32_t*)fin.gave_up);
                launch_left8(gc8, group_alloc(cnt), reinterpret_cast<const float4*>(img), (int)ntiles, fin, assign + n0,
                             dist ? dist + n0 : nullptr, st, rl);
            }
        } else if (filter) {
            if constexpr (M == 4) {
                const bool bucket = files_records && variant == 63 && N <= per_launch;
                BucketOut bo{};
                if (bucket) {
                    bo = BucketOut{reinterpret_cast<uint2*>(ws + c.pool_off), reinterpret_cast<uint2*>(ws + c.bseg_off), link->KT,
                                   link->ngroups};
                    launch_filter4_bucket(gco, group_alloc(cnt), fin, assign + n0, dist ? dist + n0 : nullptr, st, bo, &link->nwg);
                    link->produced = true;
                } else {
                    launch_filter4(variant, gco, group_alloc(cnt), fin, assign + n0, dist ? dist + n0 : nullptr, st, rl,
                                   opt.rounds_per_launch);
                }
                hipLaunchKernelGGL((tile_image_kernel<4, 2>), dim3(left_blocks), dim3(256), 0, st, centers, K, tables, img, total,
                                   reinterpret_cast<float*>(ws + c.rows_off), (const uint32_t*)fin.gave_up);
                launch_left4(gco, group_alloc(cnt), reinterpret_cast<const float4*>(img), rows, (int)ntiles, (K + 15) / 16, fin,
                             assign + n0, dist ? dist + n0 : nullptr, st, rl, bucket ? &bo : nullptr);
            }
        } else if (M == 8 && variant_two_lane(M, variant))
            launch_scan_grouped8_q(variant, gc8, group_alloc(cnt), reinterpret_cast<const float4*>(img), (int)ntiles,
                                   assign + n0, dist ? dist + n0 : nullptr, st, rl, opt.rounds_per_launch);
        else if (variant == 89 && files_records && N <= per_launch) {
            BucketOut bo{reinterpret_cast<uint2*>(ws + c.pool_off), reinterpret_cast<uint2*>(ws + c.bseg_off), link->KT,
                         link->ngroups};
            launch_scan4h_bucket(gco, group_alloc(cnt), reinterpret_cast<const float4*>(img), rows, (int)ntiles,
                                 (K + 15) / 16, assign + n0, dist ? dist + n0 : nullptr, st, bo, &link->nwg);
            link->produced = true;
        } else if (variant_lds_loads(M, variant))
            launch_scan_grouped_h(variant, gco, group_alloc(cnt), reinterpret_cast<const float4*>(img), rows, (int)ntiles,
                                  (K + 15) / 16, assign + n0, dist ? dist + n0 : nullptr, st, rl, opt.rounds_per_launch);
        else if (variant_two_lane(M, variant))
            launch_scan_grouped_q(variant, gco, group_alloc(cnt), reinterpret_cast<const float4*>(img), rows, (int)ntiles,
                                  assign + n0, dist ? dist + n0 : nullptr, st, rl, tsrc, opt.rounds_per_launch);
        else if (grouped && M == 8)
            launch_scan_grouped8(variant, gc8, group_alloc(cnt), reinterpret_cast<const float4*>(img), (int)ntiles,
                                 assign + n0, dist ? dist + n0 : nullptr, st, rl, opt.rounds_per_launch);
        else if (grouped && M == 4 && link && link->wanted && variant == 70 && N <= per_launch &&
                 c.bseg_off != c.pool_off) {
            BucketOut bo{reinterpret_cast<uint2*>(ws + c.pool_off), reinterpret_cast<uint2*>(ws + c.bseg_off), link->KT,
                         link->ngroups};
            launch_scan_grouped(variant, gco, group_alloc(cnt), reinterpret_cast<const float4*>(img), rows,
                                (int)ntiles, assign + n0, dist ? dist + n0 : nullptr, st, &bo, &link->nwg);
            link->produced = true;
        } else if (grouped)
            launch_scan_grouped(variant, gco, group_alloc(cnt), reinterpret_cast<const float4*>(img), rows,
                                (int)ntiles, assign + n0, dist ? dist + n0 : nullptr, st, nullptr, nullptr, rl);
        else
            launch_scan_M<M>(variant, codes + n0 * M, cnt, reinterpret_cast<const float4*>(img), rows, (int)ntiles,
                             assign + n0, dist ? dist + n0 : nullptr, st, left);
        if (prof) {
            hipEventRecord(ev.b, st);
            std::lock_guard<std::mutex> lk(g_mu);
            g_scan_log.kernels += t_scan_kernels > 0 ? t_scan_kernels : 1;
        }
        if (launched() != PQKM_OK) return PQKM_ERR_DEVICE;
    }
    carried = plan_of.leaves;
    return PQKM_OK;
}

// Scan with one lane per center: from this many centers on the table rows of a block's codes are copied to LDS first.
// Aligned operands, straight into LDS, us through the caches / so: M = 4, K = 1: 12.4 / 8.9 at N = 16384, K = 100: 12.9 / 9.1; M = 8, K = 16:
// 4.8 / 4.5 at N = 2000 and 9.6 / 9.6 at 1e4; M = 16, N = 1e4: 13.5 / 16.2 at K = 64, 15.0 / 16.5 at K = 80, 17.8 / 17.0 at K = 100; M = 32, N =
// 2000: 10.5 / 9.7 at K = 130.  Byte by byte, one code per block, N = 4e5, ms: M = 1, K = 2000: 0.76 / 2.07, M = 6: 1.22 / 2.17 at K =
// 500 and 4.7 / 3.8 at K = 2000, M = 24: 1.99 / 4.33 at K = 200 and 9.2 / 6.8 at K = 1000.
inline int gather_rows_min_k(int M, bool words) { return words ? (M < 16 ? 1 : M == 16 ? 96 : 160) : 250 + 6000 / M; }

// With few centers most of its lanes have none, and one lane per code (assign_generic_kernel) is faster: that takes about
// 0.27 us per look-up of a code while the codes do not fill the chip and 3.9 ps each beyond, the scan above 0.75 ns and 0.03 ns
// M per code.  Measured, one lane per code / per center, us: M = 2, K = 16: 11 / 19 at N = 2e4, 44 / 333 at 4e5; M = 6, N = 4e5:
// 138 / 445 at K = 16, 599 / 471 at 64; M = 24, N = 4e5: 169 / 950 at K = 4, 800 / 1330 at 16, 3700 / 1450 at 64.
bool lane_per_code(int64_t N, int M, int K)
{
    const double fill = 0.0033 * (double)N;
    return (double)K * M < (fill < 215.0 ? fill : 215.0) * (1.0 + M / 22.0);
}

// us of the scan with one lane per center and its rows in LDS (many codes): measured at K = 160, 300, 1000 and 4000, ns per code: M = 4:
// 0.40, 0.44, 0.85, 2.8; M = 8: 0.68, 0.79, 1.6, 5.6; M = 16: 1.35, 1.6, 3.3, 10.8; M = 32: 3.35, 3.9, 5.9, 21.  A block's only pass takes hardly less with
// fewer than 256 centers (K = 180, 200, 230: M = 4: 0.39, 0.41, 0.41; M = 8: 0.70, 0.72, 0.73).
double rows_us(int64_t N, int M, int K)
{
    const double base = M == 4 ? 0.26 : M == 8 ? 0.43 : M == 16 ? 1.0 : 2.4, pass = M == 4 ? 0.164 : M == 8 ? 0.33 : M == 16 ? 0.61 : 1.15;
    const double least = M == 4 ? 0.405 : M == 8 ? 0.725 : 0.0, code = base + pass * ((double)K / 256.0);
    return 3.6 + 0.001 * (double)N * (code > least ? code : least);
}

// us of the tiled scans while one round of their smallest workgroups covers the codes: a fixed part and the tiles of 128 / M centers
double one_round_tiled_us(int M, int K)
{
    const double tiles = (double)(((int64_t)K * M + 127) / 128);
    return M == 4 ? 8.0 + 2.45 * tiles : M == 8 ? 9.5 + 2.12 * tiles : M == 16 ? 11.8 + 2.13 * tiles : 19.5 + 2.63 * tiles;
}

// Codes up to which one lane per center is the faster one whatever the alignment
inline int64_t gather_codes_any(int K) { return (int64_t)120000 * K / (1550 + (int64_t)K); }

// Most codes for which it is faster than the tiled scans (M = 4, 8, 16, 32), whose time does not depend on N below one round of their
// smallest workgroups: a fixed part and about 2.45 us (M = 4) per tile of 128 / M centers.  Where the scan on the matrix cores takes
// over from the tiled ones (dot_scan_dims) that is the limit.  With distances, tiled / one lane per center, us, on either side: M = 4, K = 1000:
// 87 / 64 at N = 7e4, 90 / 98 at 1.1e5; K = 300: 32.6 / 22.5 at 4e4, 33 / 36 at 7e4; M = 8, K = 300: 50 / 37 at 4e4, 51 / 59 at 7e4; M = 16, K =
// 160: 55 / 33 at 2e4, 55 / 60 at 4e4; M = 32, K = 160: 136 / 73 at 2e4, 134 / 138 at 4e4.  Fewer than 160 centers: 7 us + 0.6 ns N against 7 us + 2.8 us
// for every 32 centers at M = 4, 4.7 us at M = 8 and 7 us at M = 16, the line of the rows through the caches, which hold for M = 16 below 96 centers and M =
// 32; with the rows in LDS the two are even at twice to three times as many codes: M = 4: 10.3 / 10.5 at 2e4, K = 16; 17.3 / 18.8 at 4e4, K = 100 (12.5 /
// 7.3 at 1e4, K = 64); M = 8: 13.3 / 13.5 at 16384, K = 32; 28.5 / 31.6 at 4e4, K = 130; M = 16: 39.3 / 29.8 at 2e4, K = 100.
// Centers that are not aligned are read byte by byte, one code per block, several times as slowly, and the line stays lower.  Tiled / so, us:
// M = 4, K = 1000: 88 / 431 at 9e4, K = 300: 32 / 88 at 4.6e4; M = 8, K = 1000: 145 / 562 at 7e4; M = 32, K = 300: 223 / 365 at 2.5e4.
int64_t gather_max_codes(int M, int K, bool aligned)
{
    const int64_t least = gather_codes_any(K);
    if (K >= 160 && !aligned) return least;
    if (K >= 160) {
        int64_t most = (int64_t)((one_round_tiled_us(M, K) - 3.6) / (rows_us(1000000, M, K) - 3.6) * 1e6);
        const int64_t dot_from = M == 8 ? 90000000 / K : M == 16 && 9000000 / K < 25000 ? 25000 : 9000000 / K;
        if (M > 4 && (M > 8 || K >= 500) && most >= dot_from) most = dot_from - 1;
        if (most > 512 * (int64_t)cu_count()) most = 512 * (int64_t)cu_count();
        return most > least ? most : least;
    }
    const int64_t most = (int64_t)(M == 4 ? 4700 : M == 8 ? 7800 : 11600) * ((K + 31) / 32);
    return M == 32 || most > 16384 ? 16384 : most;
}

// Is the scan on the matrix cores tried before the one with one lane per center, and for how many dimensions?  While its blocks of 256
// codes fill the chip no more than once it takes a time that hardly depends on N, more by half at 256 dimensions; tables it is not for
// cost 10 us (M = 8: 14) and are left to the scan behind, as those of 256 dimensions are where only 128 pay.  One lane per
// center alone, then this with tables of 128 / 256 dimensions / it is not for, us, with distances: M = 8, K = 1000: 57 (51 / 69 / 67) at N =
// 3.3e4, 78 (60 / 76 / 86) at 4.6e4; K = 4000: 142 (91 / 147 / 148) at 2.5e4, 251 (122 / 151 / 261) at 4.6e4; M = 16, K = 300: 45 (40 / 56 / 53) at
// 2.5e4; K = 1000: 63 (49 / 71 / 73) at 1.8e4, 152 (65 / 75 / 159) at 4.6e4; K = 4000: 201 (92 / 138 / 208) at 1.8e4; M = 32, K = 160: 90 (53 / 59 /
// 99) at 2.5e4; K = 1000: 78 (61 / 77 / 86) at 1.2e4, 279 (69 / 95 / 290) at 4.6e4.  More centers than codes lie close together, and a scan that then leaves them
// all was for nothing (M = 16, N = 8000, K = 50000 of 500 components: 1060 and 1590): it has to promise more.
// Nor where tables that it is not for would take longer than by the tiled scans, us, tiled / 128 dimensions / left to one lane per center: M = 8, K = 300: 50
// (44 / 59) at 5.6e4; K = 400: 63 (47 / 71) at 6.2e4, but K = 512: 80 (48 / 77) at 6e4; M = 16, K = 160: 55 (40 / 66) at 3.7e4; K = 200: 66 (42 / 75) at 4.2e4,
// but K = 256: 84 (40 / 67) at 3.5e4; M = 32, K = 160: 134 (51 / 147) at 3.9e4.  (rows_us is a tenth too long at M = 8 between 256 and 700 centers.)
int dot_before_rows(int M, const Options& opt, int64_t N, int K, const uint8_t* codes, const uint8_t* centers, const Carve& c)
{
    if (M < 8 || !tiled_M(M) || K < 160 || K > (1 << 22) || opt.assign_kernel == 1 || c.dot_off == 0 ||
        (((uintptr_t)codes | (uintptr_t)centers) & 3) != 0)
        return 0;
    const int64_t round = 256 * (int64_t)cu_count(), rounds = (N + round - 1) / round;
    const double few = M == 8 ? 35.0 : M == 16 ? 32.0 : 45.0, many = M == 8 ? 49.0 : M == 16 ? 37.0 : 51.0, rows = rows_us(N, M, K);
    auto dot = [&](double fixed, double center) { return fixed + center * K * (double)rounds + 10.0 * (double)(rounds - 1); };
    if (N > gather_codes_any(K) && rows + (M == 8 ? 14.0 : 10.0) > (M == 8 ? 1.12 : 1.0) * one_round_tiled_us(M, K)) return 0;
    return rows > (K > N ? 1.6 : 1.25) * dot(many, 0.025) ? 256 : rows > (K > N ? 1.5 : 1.2) * dot(few, 0.015) ? 128 : 0;
}

// does one of the LDS-tiled scans run?
bool tiled_scan(const Options& opt, int64_t N, int M, int K, const uint8_t* codes, const uint8_t* centers)
{
    if (!tiled_M(M) || opt.assign_kernel == 1 || ((uintptr_t)codes & 3) != 0) return false;
    return opt.assign_kernel != 0 || opt.scan_variant != 0 || N > gather_max_codes(M, K, ((uintptr_t)centers & 3) == 0);
}

// What the scan with one lane per center does with N codes (one lane per code where `per_code`).
struct GatherPlan {
    bool words;               // codes and centers are read as words
    bool rows;                // the rows of a block's codes are copied to LDS
    bool per_code;
    int codes;                // per block
    int64_t parts;            // that the centers are split into
};

// room: for the records of the parts; `whole`: it is in use, so that the centers stay in one part
GatherPlan gather_plan(int64_t N, int M, int K, bool aligned, size_t room, bool whole)
{
    GatherPlan p{};
    p.words = tiled_M(M) && aligned;
    p.rows = K >= gather_rows_min_k(M, p.words);
    p.codes = 1;
    p.parts = 1;
    if (!p.words && lane_per_code(N, M, K)) {
        p.per_code = true;
        return p;
    }
    const int64_t passes = ((int64_t)K + 255) / 256;               // of a block over its centers
    const int64_t ncu = cu_count(), records = (int64_t)(room / sizeof(NearRecord));
    if (p.words && p.rows) {
        // Codes per block and parts of the centers by the time they take: a compute unit has k blocks, and a block's pass takes 10 ns M per
        // code of it where they share the unit, and 20 ns more by itself; beside its passes a block costs 50 ns + 4.5 ns M per code,
        // and parts a second launch.  What matters is how evenly the blocks fill the units.  us, codes x parts: M = 4, N = 257, K = 300000:
        // 122 (1 x 1) / 60 (1 x 16); N = 1025: 393 (4 x 1) / 213 (2 x 12); N = 2100, K = 50000: 103 (4 x 1) / 77 (2 x 6); N = 500, K =
        // 1000: 4.2 (1 x 1) / 4.3 (2 x 1) / 4.9 (4 x 1), N = 8000: 12.6 / 10.6 / 10.0; M = 8, N = 257, K = 300000: 196 / 110 (1 x 24);
        // M = 16, N = 257, K = 50000: 69 / 42 (2 x 16), N = 8000, K = 1000: 30.1 (1 x 1) / 28.6 (2 x 1) / 33.5 (4 x 1); M = 32, N =
        // 257, K = 50000: 134 / 79 (1 x 24).  Two codes of M = 16 leave room for fewer blocks, which few passes show: K = 300, N = 1e4: 19.4 / 21.7.
        // (A block of one code per unit and too few passes for parts: nothing to choose, and the call waits for this arithmetic.)
        if (N <= ncu && (double)passes * (M < 8 ? 0.09 : 0.0104 * M + 0.02) < 2.8) return p;
        double best = 1e300;
        const int widest = N < 2 || M == 32 || (M == 16 && passes <= 2) ? 1 : M == 4 ? 4 : 2;
        for (int log = 0; 1 << log <= widest; ++log) {
            const int codes = 1 << log;
            const int64_t blocks = (N + codes - 1) >> log;
            const double code = 0.0104 * M * codes, pass = code + (codes == 1 ? 0.005 : 0.0), lone = code + 0.02 < 0.09 ? 0.09 : code + 0.02;
            const double beside = 0.05 + 0.0045 * M * codes;
            const int64_t parts_of[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 64, 128, passes};
            for (int64_t parts : parts_of) {
                if (parts > 1 && (whole || (double)passes * lone < 2.8)) break;
                if (parts > 1 && (parts > passes || parts * N > records || parts > 128)) continue;
                const double mine = (double)(parts == 1 ? passes : (passes + parts - 1) / parts), k = (double)((blocks * parts + ncu - 1) / ncu);
                const double one = mine * lone + beside, all = k * (mine * pass + beside);
                const double us = (one > all ? one : all) + (parts > 1 ? 2.8 + 0.0006 * (double)N : 0.0);
                if (us < best) { best = us; p.codes = codes; p.parts = parts; }
            }
        }
        return p;
    }
    // about eight blocks per compute unit, as long as each keeps 256 centers
    if (whole || N < 1) return p;
    p.parts = 8 * ncu / N;
    if (p.parts > passes) p.parts = passes;
    if (p.parts * N > records) p.parts = records / N;
    if (p.parts < 1) p.parts = 1;
    return p;
}

template <int MW, int CN>
pqkm_status launch_gather(const GatherPlan& plan, const uint8_t* codes, int64_t N, int M, const uint8_t* centers, int K, const float* tables,
                          int32_t* assign, float* dist, NearRecord* part, const DotState* front, hipStream_t st)
{
    const int64_t per_launch = (int64_t)CN << 23;                  // 2^31 threads
    for (int64_t n0 = 0; n0 < N; n0 += per_launch) {
        const int64_t cnt = N - n0 < per_launch ? N - n0 : per_launch;
        const int64_t blocks = (cnt + CN - 1) / CN;
        int64_t splits = plan.parts;
        int per = K;
        if (splits > 1) {
            per = (int)((((int64_t)K + splits - 1) / splits + 255) / 256 * 256);
            splits = ((int64_t)K + per - 1) / per;
        }
        if (splits < 1) splits = 1;
        float* dn = dist ? dist + n0 : nullptr;
        NearRecord* pn = splits > 1 ? part : nullptr;
        const dim3 grid((unsigned)blocks, (unsigned)splits);
        ++t_scan_kernels;
        auto launch_rows = [&]() {
            if constexpr (MW > 0)
                hipLaunchKernelGGL((assign_rows_kernel<MW, CN>), grid, dim3(256), 0, st, codes + n0 * M, cnt, centers, K, tables, assign + n0,
                                   dn, pn, per, front ? &front->left : nullptr, front ? &front->some : nullptr);
            else
                hipLaunchKernelGGL((assign_gather_kernel<0, true>), grid, dim3(256), 0, st, codes + n0 * M, M, centers, K, tables, assign + n0,
                                   dn, pn, per);
        };
        // through the caches: byte by byte, or few centers from sixteen subspaces on (gather_rows_min_k), one code per block
        if constexpr (CN == 1 && (MW == 0 || MW >= 4)) {
            if (plan.rows)
                launch_rows();
            else
                hipLaunchKernelGGL((assign_gather_kernel<MW, false>), grid, dim3(256), 0, st, codes + n0 * M, M, centers, K, tables, assign + n0,
                                   dn, pn, per);
        } else {
            launch_rows();
        }
        if (splits > 1)
            hipLaunchKernelGGL(assign_merge_kernel, dim3((unsigned)((cnt + 3) / 4)), dim3(256), 0, st, pn, cnt, (int)splits,
                               assign + n0, dn);
    }
    return launched();
}

// one lane per center, or per code where there are few centers; `front`: state of the scan on the matrix cores that was tried first
pqkm_status assign_untiled(const Carve& c, const uint8_t* codes, int64_t N, int M, const uint8_t* centers, int K,
                           const float* tables, int32_t* assign, float* dist, void* ws, const DotState* front, hipStream_t st)
{
    NearRecord* part = tiled_M(M) ? reinterpret_cast<NearRecord*>(static_cast<char*>(ws) + c.img_off) : nullptr;
    const GatherPlan p = gather_plan(N, M, K, (((uintptr_t)codes | (uintptr_t)centers) & 3) == 0, tiled_M(M) ? c.img_bytes : 0, front != nullptr);
    if (p.per_code) {
        hipLaunchKernelGGL(assign_generic_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, codes, N, M, centers, K,
                           tables, assign, dist);
        return launched();
    }
    if (p.words && M == 4 && p.codes == 1) return launch_gather<1, 1>(p, codes, N, M, centers, K, tables, assign, dist, part, front, st);
    if (p.words && M == 4 && p.codes == 2) return launch_gather<1, 2>(p, codes, N, M, centers, K, tables, assign, dist, part, front, st);
    if (p.words && M == 4) return launch_gather<1, 4>(p, codes, N, M, centers, K, tables, assign, dist, part, front, st);
    if (p.words && M == 8 && p.codes == 1) return launch_gather<2, 1>(p, codes, N, M, centers, K, tables, assign, dist, part, front, st);
    if (p.words && M == 8) return launch_gather<2, 2>(p, codes, N, M, centers, K, tables, assign, dist, part, front, st);
    if (p.words && M == 16 && p.codes == 2) return launch_gather<4, 2>(p, codes, N, M, centers, K, tables, assign, dist, part, front, st);
    if (p.words && M == 16) return launch_gather<4, 1>(p, codes, N, M, centers, K, tables, assign, dist, part, front, st);
    if (p.words && M == 32) return launch_gather<8, 1>(p, codes, N, M, centers, K, tables, assign, dist, part, front, st);
    return launch_gather<0, 1>(p, codes, N, M, centers, K, tables, assign, dist, part, front, st);
}

pqkm_status assign_core(const Options& opt, const Carve& c, const uint8_t* codes, int64_t N, int M,
                        const uint8_t* centers, int K, const float* tables, int32_t* assign, float* dist, void* ws,
                        hipStream_t st, Carried& carried, BucketLink* link)
{
    if (opt.assign_kernel == 2 && !(tiled_M(M) && ((uintptr_t)codes & 3) == 0)) return PQKM_ERR_SHAPE;
    if (!tiled_scan(opt, N, M, K, codes, centers)) {
        // tables that the scan on the matrix cores is not for are left to the one with one lane per center
        const int dims = dot_before_rows(M, opt, N, K, codes, centers, c);
        const DotState* state = nullptr;
        if (dims) {
            char* wsc = static_cast<char*>(ws);
            if (M == 8) launch_dot<8, true>(codes, N, centers, K, tables, assign, dist, c, wsc, carried, opt, dims, st);
            else if (M == 16) launch_dot<16, true>(codes, N, centers, K, tables, assign, dist, c, wsc, carried, opt, dims, st);
            else launch_dot<32, true>(codes, N, centers, K, tables, assign, dist, c, wsc, carried, opt, dims, st);
            if (launched() != PQKM_OK) return PQKM_ERR_DEVICE;
            state = reinterpret_cast<const DotState*>(wsc + c.dot_off);
            ++carried.iteration;
            carried.dot = true;
        }
        EventPair ev{};
        const bool prof = (opt.profile & 1) && log_begin(g_scan_log, st, &ev);
        t_scan_kernels = 0;
        const pqkm_status s = assign_untiled(c, codes, N, M, centers, K, tables, assign, dist, ws, state, st);
        if (prof) {
            hipEventRecord(ev.b, st);
            std::lock_guard<std::mutex> lk(g_mu);
            g_scan_log.kernels += t_scan_kernels > 0 ? t_scan_kernels : 1;
        }
        return s;
    }
    float* img = reinterpret_cast<float*>(static_cast<char*>(ws) + c.img_off);
    char* wsc = static_cast<char*>(ws);
    switch (M) {
        case 4: return assign_tiled<4>(codes, N, centers, K, tables, assign, dist, img, opt, c, wsc, carried, st, link);
        case 8: return assign_tiled<8>(codes, N, centers, K, tables, assign, dist, img, opt, c, wsc, carried, st, link);
        case 16: return assign_tiled<16>(codes, N, centers, K, tables, assign, dist, img, opt, c, wsc, carried, st, link);
        default: return assign_tiled<32>(codes, N, centers, K, tables, assign, dist, img, opt, c, wsc, carried, st, link);
    }
}

// one whole assignment step (tile images, regrouping where it is due, scan launches), optionally bracketed by events
pqkm_status assign_impl(const Options& opt, const Carve& c, const uint8_t* codes, int64_t N, int M,
                        const uint8_t* centers, int K, const float* tables, int32_t* assign, float* dist, void* ws,
                        hipStream_t st, Carried* carried = nullptr, BucketLink* link = nullptr)
{
    if (N == 0) return PQKM_OK;
    Carried none;
    none.alone = true;
    EventPair ev{};
    const bool prof = (opt.profile & 2) && log_begin(g_step_log, st, &ev);
    const pqkm_status s = assign_core(opt, c, codes, N, M, centers, K, tables, assign, dist, ws, st, carried ? *carried : none, link);
    if (prof) hipEventRecord(ev.b, st);
    return s;
}

template <int PER>
void launch_seg_scatter(const int32_t* assign, int64_t N, int K, const SegKey& sk, const uint32_t* start, uint32_t* cursor, uint32_t* sidx,
                        const SegZero& z, hipStream_t st)
{
    const unsigned blocks = (unsigned)((N + 1024 * PER - 1) / (1024 * PER));
    if (K <= 8192)
        hipLaunchKernelGGL((seg_scatter_block_kernel<PER, 8192>), dim3(blocks + (unsigned)z.groups), dim3(1024), 0, st, assign, N, K,
                           sk, start, cursor, sidx, blocks, z);
    else
        hipLaunchKernelGGL((seg_scatter_block_kernel<PER, SEG_BLOCK_MAX_K>), dim3(blocks + (unsigned)z.groups), dim3(1024), 0, st,
                           assign, N, K, sk, start, cursor, sidx, blocks, z);
}

// counting sort of the code indices by cluster, or by group of KT clusters, into the workspace: start[0..K] and sidx[0..#valid); and
// seg_zero for every group
void sort_by_cluster(const int32_t* assign, int64_t N, int K, const Carve& c, char* ws, uint32_t** start_out,
                     uint32_t** sidx_out, hipStream_t st, bool ranked = false, const SegZero& z = SegZero{}, int KT = 1, int bits = 32)
{
    // sorted by group of KT clusters, K is the number of groups from here on
    const SegKey sk{(uint32_t)K, (uint32_t)KT, KT > 1 ? (uint32_t)(((uint64_t)1 << 32) / (uint32_t)KT) + 1u : 0u, bits};
    const size_t seg_stride = align256(((size_t)K + 1) * sizeof(uint32_t));
    K = (K + KT - 1) / KT;
    uint32_t* sidx = reinterpret_cast<uint32_t*>(ws + c.sidx_off);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(ws + c.seg_off);
    uint32_t* start = reinterpret_cast<uint32_t*>(ws + c.seg_off + seg_stride);
    uint32_t* cursor = reinterpret_cast<uint32_t*>(ws + c.seg_off + 2 * seg_stride);
    unsigned sb = (unsigned)((N + 1023) / 1024 < 8192 ? (N + 1023) / 1024 : 8192);
    if (sb < 1) sb = 1;
    if (ranked) {
        // the scan of this iteration counted the clusters and left every code's rank: prefix, then place
        const uint32_t* rank = reinterpret_cast<const uint32_t*>(ws + c.rank_off);
        hipLaunchKernelGGL(seg_prefix_kernel, dim3(1), dim3(1024), 0, st, cnt, K, start, cursor);
        hipLaunchKernelGGL(seg_place_kernel, dim3(sb), dim3(256), 0, st, assign, rank, N, K, start, sidx);
        if (z.groups > 0) hipLaunchKernelGGL(seg_zero_kernel, dim3((unsigned)z.groups), dim3(256), 0, st, z, start);
        *start_out = start;
        *sidx_out = sidx;
        return;
    }
    unsigned zb = (unsigned)((K + 255) / 256 < 1024 ? (K + 255) / 256 : 1024);
    hipLaunchKernelGGL(zero_u32_kernel, dim3(zb), dim3(256), 0, st, cnt, (int64_t)K);
    // 8192 codes or more per workgroup: every one adds its K sizes to the sums
    unsigned cb = (unsigned)((N + 8191) / 8192 < 512 ? (N + 8191) / 8192 : 512);
    if (cb < 1) cb = 1;
    hipLaunchKernelGGL(seg_count_kernel, dim3(cb), dim3(1024), 0, st, assign, N, K, sk, cnt);
    hipLaunchKernelGGL(seg_prefix_kernel, dim3(1), dim3(1024), 0, st, cnt, K, start, cursor);
    if (K <= SEG_BLOCK_MAX_K) {
        // about one block per compute unit: fewer leave some idle, more pay for K more sizes each
        const int64_t per = (N + 1023) / 1024 / cu_count();
        if (per < 2) launch_seg_scatter<2>(assign, N, K, sk, start, cursor, sidx, z, st);
        else if (per < 4) launch_seg_scatter<4>(assign, N, K, sk, start, cursor, sidx, z, st);
        else if (per < 8) launch_seg_scatter<8>(assign, N, K, sk, start, cursor, sidx, z, st);
        else launch_seg_scatter<16>(assign, N, K, sk, start, cursor, sidx, z, st);
    } else {
        hipLaunchKernelGGL(seg_scatter_kernel, dim3(sb), dim3(256), 0, st, assign, N, sk, start, cursor, sidx);
        if (z.groups > 0) hipLaunchKernelGGL(seg_zero_kernel, dim3((unsigned)z.groups), dim3(256), 0, st, z, start);
    }
    *start_out = start;
    *sidx_out = sidx;
}

// what a fused iteration asks of its assignment step: records by cluster group, when the histogram would
// otherwise take the owner path (M = 4)
BucketLink bucket_request(const Options& opt, int64_t N, int M, int K)
{
    BucketLink l;
    if (N < 1) return l;
    const HistPlan hp = hist_plan(N, M, K);
    const int force = opt.hist_kernel;
    // Sorted-path sizes: the scan counts the clusters and leaves every code's rank.  Not where the owner path is possible and the sorted
    // one only faster: there the keys of the lower-bound scans lie in the ranks' room.
    if (force == 0 && !owner_histogram(hp, force) && N <= (int64_t)0xffffffff) l.rank_wanted = true;
    if (M != 4) return l;
    if (force != 0 || !owner_histogram(hp, force)) return l;     // a forced histogram kernel is used as named
    l.wanted = true;
    l.KT = hp.KT;
    l.ngroups = (int)hp.groups;
    return l;
}

// Does the vote count its histograms itself, from all codes?  Every workgroup (16 clusters of a subspace) reads all assignments and a
// byte of every code, which saves two launches.  Whole update, histogram first / so, us: M = 4: 19.5 / 14.4 at N = 1e4, K = 100, 28.7 / 22.0
// at 4e4, 1000, 25.4 / 29.3 at 8e4, 100; M = 8: 36.9 / 30.8 at 2e4, 1000, 41.2 / 41.7 at 4e4, 1000; M = 16: 26.9 / 22.5 at 2e4, 100,
// 31.6 / 32.5 at 4e4, 100, 54.7 / 60.1 at 2e4, 1000; M = 32: 33.4 / 25.7 at 1e4, 100, 45.9 / 50.8 at 1e4, 300.
inline bool vote_counts_codes(int64_t N, int M, int K)
{
    const int64_t blocks = (int64_t)((K + VOTE_REC_KT - 1) / VOTE_REC_KT) * M;
    if (M > 8) return N >= 1 && N <= 20000 && blocks <= 256;
    return N >= 1 && N <= 40000 && blocks <= (N <= 20000 ? 512 : 256);
}

// Few clusters: rows straight from the L2 (vote_few_kernel), while they are fewer than 550000 in all, from M = 4 on 524288 (a cluster has at most 256 non-zero
// bins per subspace, and no more than it has members; a workgroup's waves beyond M are idle but there).  Whole update at 4e5 codes, vote_kernel / this, us, on
// either side: M = 4: 40.3 / 36.4 at K = 488, 40.6 / 41.3 at 536; M = 5: 45.8 / 42.6 at 244, 46.2 / 49.4 at 268; M = 8: 44.4 / 41.0 and 45.1 / 47.5; M = 3: 40.5 /
// 37.5 at 714.  The vote alone, vote_kernel / this, us: M = 4: 13.1 / 6.9 at N =
// 1e4, K = 100, 23.4 / 13.5 at 1.28e6, 100, 21.0 / 17.8 at 2e5, 300, but 16.8 / 20.7 at 2e5, 1000; M = 8: 23.5 / 21.8 at 1e6, 256, but 21.2 / 24.1
// at 2e5, 300; M = 16: 19.6 / 15.8 at 4e4, 100; M = 32: 45 / 32 at 1e4, 1000.  Whole update: M = 6: 45 / 49 at 3e5, 300.
// Many rows with few bins each: where vote_kernel's workgroups of sixteen clusters are one round that is nearly full, it is the better one
// (M = 4, K = 1000: 33.7 / 35.9 at 1e5, 31 / 31 at 5e4; M = 8, K = 500: 33.4 / 35.7 at 5e4), and beyond some 10000 workgroups of this one
// their own cost shows: M = 8, K = 5000: 73 / 68 at 1e4, K = 10000: 108 / 110 at 2e4; M = 16, K = 3000: 73 / 79 at 1e4; M = 24, K = 1500: 79 / 69
// and K = 2000: 77 / 80 at 5000; M = 32, K = 1000: 61 / 56, K = 3000: 116 / 129 at 1e4; M = 64, K = 1000: 101 / 93, K = 1500: 125 / 127 at 5000; M = 6, K = 3000: 44 / 41, K = 4000: 45 / 48 at 1e4.
inline bool vote_few(int64_t N, int M, int K)
{
    const int64_t quads = (M + 3) / 4, waves = M <= 4 ? M : 4 * quads;
    const int64_t rows = (int64_t)K * waves * L < N * waves ? (int64_t)K * waves * L : N * waves;
    const int64_t kept = (int64_t)K * M / 16;                      // workgroups of vote_kernel
    if (kept > cu_count() * 2 / 3 && kept <= cu_count() && rows > 190000) return false;
    const int64_t most = M <= 3 ? 550000 : (int64_t)2 * cu_count() * 4 * L;       // two rounds of its workgroups with all bins
    return N >= 1 && rows <= most && (int64_t)K * quads <= (M <= 4 ? 10000 : M % 4 ? 6000 : M <= 8 ? 10000 : M < 40 ? 9000 : 250 * M);
}

// Few codes as well: each of its workgroups counts its cluster from all codes, as few subspaces as one round of them allows.  Whole update, us,
// where vote_kernel counts or a histogram is formed first / so: M = 4: 17 / 10 at N = 1e4, K = 100, 27.3 / 18.2 at 2e4, 32, 18.0 / 13.2 at 2e4, 256,
// 31.0 / 24.3 at 4e4, 64, 24.7 / 20.3 at 4e4, 256, but 31.8 / 35.0 at 8e4, 100; M = 8: 20.9 / 16.5 at 2e4, 128, 31.1 / 27.2 at 4e4, 64; M = 16: 34.3 /
// 29.1 at 4e4, 64.  A workgroup with a large share of the codes takes longer: 23.4 / 22.8 at 3e4, 8, but 25.2 / 26.6 at 4e4, 8 and 37.8 / 46.2 at
// M = 64; the vote itself 19.8 / 18.8 at 19084, 2, but 20.3 / 21.5 at 24550, 3.  Byte by byte, four subspaces are too many: M = 6: 20.4 / 16.5 at 12000, 64, but 17.0 / 17.9 at 12000, 128.  All codes in one cluster:
// M = 4: 19.6 / 18.3 at 2e4, 64, 19.8 / 21.4 at 2e4, 256, 23.1 / 26.0 at 4e4, 64; all of them alike: 26 / 17 at 2e4, 64 (70 in one copy of the bins).
// Returns the subspaces per workgroup, 0: not.
inline int vote_few_counts_codes(int64_t N, int M, int K, const uint8_t* codes)
{
    const bool words = (M & 3) == 0 && ((uintptr_t)codes & 3) == 0;
    if (N < 1 || N > (!words ? 12000 : K < 4 ? 20000 : K < 16 ? 28000 : 40000)) return 0;
    for (int G = 1; G <= (words || N < 1500 ? 4 : 2); G *= 2)
        if ((int64_t)K * ((M + G - 1) / G) <= cu_count()) return G;
    return 0;
}

// How an update counts its histograms: as hist_path says, or the vote counts them itself, a workgroup per cluster and four subspaces or
// per sixteen clusters and one (not where the scan has left records).
enum UpdateRoute { UPDATE_PASS, UPDATE_IN_VOTE_FEW, UPDATE_IN_VOTE };
UpdateRoute update_route(HistPath path, int force, int64_t N, int M, int K, const uint8_t* codes)
{
    if (path == HIST_RECORDS || force != 0) return UPDATE_PASS;
    if (vote_few_counts_codes(N, M, K, codes)) return UPDATE_IN_VOTE_FEW;
    return vote_counts_codes(N, M, K) ? UPDATE_IN_VOTE : UPDATE_PASS;
}

pqkm_status update_impl(const Options& opt, const Carve& c, const uint8_t* codes, int64_t N, int M,
                        const int32_t* assign, int K, const float* tables, uint8_t* centers, uint32_t* hist,
                        uint32_t* counts, void* ws, hipStream_t st, const BucketLink* link = nullptr)
{
    if (!hist) hist = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + c.hist_off);
    if (!counts) counts = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + c.counts_off);
    const int64_t nh = (int64_t)K * M * L;
    auto zero_hist = [&]() {
        unsigned zb = (unsigned)((nh + 255) / 256 < 65536 ? (nh + 255) / 256 : 65536);
        hipLaunchKernelGGL(zero_u32_kernel, dim3(zb), dim3(256), 0, st, hist, nh);
    };
    // Owner path (LDS-privatised, no global atomics) while streaming the assignment array once per cluster
    // group is cheap; otherwise one global atomic per code and subspace into a zeroed histogram.
    const HistPlan hp = hist_plan(N, M, K);
    const int force = opt.hist_kernel;
    int S = 1;
    bool halves = false;
    size_t part_stride = 0;
    uint32_t* parts = hist;
    const HistPath path = hist_path(N, M, K, c, force, link && link->produced && link->KT == hp.KT && link->ngroups == (int)hp.groups,
                                    link && scans_keep_keys(M));
    const bool linked = path == HIST_RECORDS;
    if (linked && M == 4 && hp.KT <= VOTE_REC_KT && link->nwg <= VOTE_REC_SEGS) {
        // the scan of this iteration filed (code, center) records by cluster group, and a vote workgroup can take
        // one group (and one subspace): it counts its histograms itself -- no histogram pass at all
        const uint2* pool = reinterpret_cast<const uint2*>(static_cast<char*>(ws) + c.pool_off);
        const uint2* bseg = reinterpret_cast<const uint2*>(static_cast<char*>(ws) + c.bseg_off);
        hipLaunchKernelGGL((vote_kernel<VOTE_RECORDS>), dim3((unsigned)(hp.groups * M)), dim3(VOTE_THREADS), 0, st, hist, hist, 1,
                           (size_t)0, counts, K, M, hp.KT, tables, centers, VoteRecords{pool, bseg, link->nwg, nullptr, nullptr, 0});
        return launched();
    }
    const UpdateRoute route = update_route(path, force, N, M, K, codes);
    if (route == UPDATE_IN_VOTE_FEW) {
        const int G = vote_few_counts_codes(N, M, K, codes);
        const dim3 grid((unsigned)((int64_t)K * ((M + G - 1) / G)));
        const VoteRecords all{nullptr, nullptr, 0, codes, assign, N};
        if (G == 1)
            hipLaunchKernelGGL((vote_few_kernel<VOTE_CODES, 1>), grid, dim3(VOTE_FEW_THREADS), 0, st, hist, hist, 1, (size_t)0, false, counts, K, M, tables, centers, all);
        else if (G == 2)
            hipLaunchKernelGGL((vote_few_kernel<VOTE_CODES, 2>), grid, dim3(VOTE_FEW_THREADS), 0, st, hist, hist, 1, (size_t)0, false, counts, K, M, tables, centers, all);
        else
            hipLaunchKernelGGL((vote_few_kernel<VOTE_CODES, 4>), grid, dim3(VOTE_FEW_THREADS), 0, st, hist, hist, 1, (size_t)0, false, counts, K, M, tables, centers, all);
        return launched();
    }
    if (route == UPDATE_IN_VOTE) {
        hipLaunchKernelGGL((vote_kernel<VOTE_CODES>), dim3((unsigned)(((K + VOTE_REC_KT - 1) / VOTE_REC_KT) * M)), dim3(VOTE_THREADS), 0, st,
                           hist, hist, 1, (size_t)0, counts, K, M, VOTE_REC_KT, tables, centers,
                           VoteRecords{nullptr, nullptr, 0, codes, assign, N});
        return launched();
    }
    if (linked) {
        // the scan of this iteration filed (code, center) records by cluster group: count from those
        S = hp.S;
        if (S > 1) {
            parts = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + c.parts_off);
            part_stride = align256(c.hist_bytes) / sizeof(uint32_t);
        }
        const uint2* pool = reinterpret_cast<const uint2*>(static_cast<char*>(ws) + c.pool_off);
        const uint2* bseg = reinterpret_cast<const uint2*>(static_cast<char*>(ws) + c.bseg_off);
        if ((int64_t)hp.KT * M * L <= HIST_LDS_WORDS_SMALL)
            hipLaunchKernelGGL((histogram_bucket_kernel<HIST_LDS_WORDS_SMALL>), dim3((unsigned)(hp.groups * S)),
                               dim3(1024), 0, st, pool, bseg, link->nwg, K, hp.KT, S, parts, part_stride);
        else
            hipLaunchKernelGGL((histogram_bucket_kernel<HIST_LDS_WORDS>), dim3((unsigned)(hp.groups * S)), dim3(1024),
                               0, st, pool, bseg, link->nwg, K, hp.KT, S, parts, part_stride);
    } else if (path == HIST_SUBSPACE) {
        const SubspaceHist sh = subspace_hist(N, M, K, c);
        S = sh.S;
        if (S > 1) {
            parts = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + c.sidx_off);
            part_stride = align256((size_t)nh * (sh.halves ? sizeof(uint16_t) : sizeof(uint32_t))) / sizeof(uint32_t);
        }
        halves = sh.halves;
        const dim3 grid((unsigned)((M + sh.G - 1) / sh.G * S));
        if (halves)
            hipLaunchKernelGGL((histogram_subspace_kernel<true>), grid, dim3(1024), 0, st, codes, N, M, assign, K, sh.G, S, parts, part_stride);
        else
            hipLaunchKernelGGL((histogram_subspace_kernel<false>), grid, dim3(1024), 0, st, codes, N, M, assign, K, sh.G, S, parts, part_stride);
    } else if (path == HIST_OWNER) {
        S = hp.S;
        if (S > 1) {
            parts = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + c.parts_off);
            part_stride = align256(c.hist_bytes) / sizeof(uint32_t);
        }
        uint8_t* gid = reinterpret_cast<uint8_t*>(static_cast<char*>(ws) + c.gid_off);
        if (N > 0)
            hipLaunchKernelGGL(cluster_group_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, assign, N, K,
                               hp.KT, gid);
        if ((int64_t)hp.KT * M * L <= HIST_LDS_WORDS_SMALL)
            hipLaunchKernelGGL((histogram_owner_kernel<HIST_LDS_WORDS_SMALL>), dim3((unsigned)(hp.groups * S)),
                               dim3(1024), 0, st, codes, N, M, assign, gid, K, hp.KT, S, parts, part_stride);
        else
            hipLaunchKernelGGL((histogram_owner_kernel<HIST_LDS_WORDS>), dim3((unsigned)(hp.groups * S)), dim3(1024),
                               0, st, codes, N, M, assign, gid, K, hp.KT, S, parts, part_stride);
    } else if (path == HIST_SORTED) {
        // sorted path: counting sort of the code indices by cluster, then LDS histograms per stretch of clusters
        uint32_t *start, *sidx;
        // 64 KB of counters per workgroup, two workgroups per compute unit: half the grain of a round (128 KB: 1.04 to 1.16 times the
        // update at M = 4, 6, 8, 16).  From M = 32 on that is one or two clusters, and with few codes in each the workgroups' own cost
        // shows: M = 48, N = 3e5, K = 1500: 301 us against 282 with 128 KB where they are even, 277 against 307 where they are tight.
        const int hist_words = M < 32 || N >= (int64_t)200 * K ? SEG_HIST_WORDS : HIST_LDS_WORDS;
        int KT = (hist_words / L) / M;
        if (KT > 128) KT = 128;
        // groups of more than twice the average of codes are shared by several workgroups
        const int64_t ng = ((int64_t)K + KT - 1) / KT;
        const int64_t twice = 2 * ((N + ng - 1) / ng);
        const uint32_t most = (uint32_t)(twice > 8192 ? (twice < 0x40000000 ? twice : 0x40000000) : 8192);
        // further shares: at most half as many as groups, listed in the room of the cluster sizes, which are not needed any more
        const int64_t further = ng > 1 ? N / most : 0;
        const size_t seg_stride = align256(((size_t)K + 1) * sizeof(uint32_t));
        uint2* items = reinterpret_cast<uint2*>(static_cast<char*>(ws) + c.seg_off);
        uint32_t* cursor = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + c.seg_off + 2 * seg_stride);
        // Sorted by group only, where the scan has not left ranks and a place in the group fits beside the index: as many
        // counters as groups in the sort, longer stretches of a block's codes in its stores, no search for the cluster.
        const bool ranked = link && link->ranked;
        int bits = 32;
        while ((KT - 1) >> (32 - bits)) --bits;
        if (ranked || KT == 1 || N > ((int64_t)1 << bits) || K > (1 << 24)) bits = 32;
        uint32_t* const listed = cursor + (bits < 32 ? ng : K);        // behind the keys' cursors
        sort_by_cluster(assign, N, K, c, static_cast<char*>(ws), &start, &sidx, st, ranked,
                        further > 0 ? SegZero{(int)ng, M, K, KT, bits < 32 ? 1 : KT, most, hist, listed, items} : SegZero{},
                        bits < 32 ? KT : 1, bits);
        if (hist_words == SEG_HIST_WORDS)
            hipLaunchKernelGGL((seg_hist_kernel<SEG_HIST_WORDS>), dim3((unsigned)(ng + further)), dim3(1024), 0, st, codes, M, bits, start, sidx, K, KT,
                               further > 0 ? most : 0xffffffffu, (int)ng, listed, items, hist);
        else
            hipLaunchKernelGGL((seg_hist_kernel<HIST_LDS_WORDS>), dim3((unsigned)(ng + further)), dim3(1024), 0, st, codes, M, bits, start, sidx, K, KT,
                               further > 0 ? most : 0xffffffffu, (int)ng, listed, items, hist);
    } else {
        zero_hist();
        const int64_t per = (int64_t)1 << 30;
        for (int64_t n0 = 0; n0 < N; n0 += per) {
            int64_t cnt = N - n0 < per ? N - n0 : per;
            hipLaunchKernelGGL(histogram_atomic_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st,
                               codes + n0 * M, cnt, M, assign + n0, K, hist);
        }
    }
    // vote_kernel adds at most 16 partial arrays, of 32-bit counters
    if (path == HIST_SUBSPACE || vote_few(N, M, K)) {
        hipLaunchKernelGGL((vote_few_kernel<VOTE_PARTS>), dim3((unsigned)(((int64_t)K + 7) / 8 * 8 * ((M + 3) / 4))), dim3(256), 0, st, hist, parts, S, part_stride,
                           halves, counts, K, M, tables, centers, VoteRecords{});
        return launched();
    }
    // vote: one workgroup per (subspace, CW clusters); about a thousand workgroups, at least one cluster per wave
    int64_t cw = ((int64_t)K * M + 1023) / 1024;
    cw = ((cw + 15) / 16) * 16;
    constexpr int vote_pass = VOTE_WAVES * VOTE_CPW;
    if (cw > 16) cw = ((cw + vote_pass - 1) / vote_pass) * vote_pass;   // whole passes of the waves
    if (cw > VOTE_MAX_CW) cw = VOTE_MAX_CW;
    const int64_t blocks_per_m = ((int64_t)K + cw - 1) / cw;
    hipLaunchKernelGGL((vote_kernel<VOTE_PARTS>), dim3((unsigned)(blocks_per_m * M)), dim3(VOTE_THREADS), 0, st, hist, parts, S,
                       part_stride, counts, K, M, (int)cw, tables, centers, VoteRecords{});
    return launched();
}

// workspace of the indexed assignment: sorted rows of A^0 and A^1, row minima, bucket counters / starts / cursors, items
struct IndexCarve { size_t ord_off, rowmin_off, cnt_off, start_off, cursor_off, items_off, total; };

IndexCarve index_carve(int M, int K)
{
    IndexCarve c{};
    size_t off = 0;
    c.ord_off = off;     off += align256((size_t)2 * L * L);
    c.rowmin_off = off;  off += align256((size_t)M * L * sizeof(float));
    c.cnt_off = off;     off += align256((size_t)(INDEX_BUCKETS + 1) * sizeof(uint32_t));
    c.start_off = off;   off += align256((size_t)(INDEX_BUCKETS + 1) * sizeof(uint32_t));
    c.cursor_off = off;  off += align256((size_t)(INDEX_BUCKETS + 1) * sizeof(uint32_t));
    c.items_off = off;   off += align256((size_t)K * sizeof(uint32_t));
    c.total = off;
    return c;
}

// BuildTable + FindNN of Alg. 1 with the table: files the centers, then one lane per code walks the buckets
pqkm_status assign_indexed_impl(const IndexCarve& c, const uint8_t* codes, int64_t N, int M, const uint8_t* centers, int K,
                                const float* tables, int32_t* assign, float* dist, char* ws, hipStream_t st)
{
    uint8_t* ord = reinterpret_cast<uint8_t*>(ws + c.ord_off);
    float* rowmin = reinterpret_cast<float*>(ws + c.rowmin_off);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(ws + c.cnt_off);
    uint32_t* start = reinterpret_cast<uint32_t*>(ws + c.start_off);
    uint32_t* cursor = reinterpret_cast<uint32_t*>(ws + c.cursor_off);
    uint32_t* items = reinterpret_cast<uint32_t*>(ws + c.items_off);
    hipLaunchKernelGGL(index_rows_kernel, dim3(L, (unsigned)M), dim3(256), 0, st, tables, ord, rowmin);
    hipLaunchKernelGGL(zero_u32_kernel, dim3(64), dim3(256), 0, st, cnt, (int64_t)INDEX_BUCKETS);
    hipLaunchKernelGGL(index_count_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, centers, K, M, cnt);
    hipLaunchKernelGGL(seg_prefix_kernel, dim3(1), dim3(1024), 0, st, cnt, INDEX_BUCKETS, start, cursor);
    hipLaunchKernelGGL(index_scatter_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, centers, K, M, start,
                       cursor, items);
    if (N > 0)
        hipLaunchKernelGGL(assign_indexed_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, codes, N, M, centers,
                           tables, ord, rowmin, start, items, assign, dist);
    return launched();
}

// Encoder: a workgroup holds the split codewords of G subspaces, as many as fit 128 KB of LDS, so that it reads whole
// stretches of the vectors; with few vectors one subspace per workgroup, so that more workgroups share the work.
template <int DP, int THREADS>
void launch_encode(const float* vectors, int64_t N, int M, int Ds, const float* codewords, uint8_t* codes, hipStream_t st)
{
    constexpr int WAVES = THREADS / 64, KS = DP <= 16 ? 1 : DP / 16;
    int G = 8 / KS;
    if (G > M) G = M;
    const int64_t tiles = (N + 31) / 32;
    const int64_t ncu = cu_count();
    auto groups = [&](int g) { return (int64_t)((M + g - 1) / g); };
    while (G > 1 && groups(G) * ((tiles + WAVES - 1) / WAVES) < ncu) G = (G + 1) / 2;
    int64_t wpg = (tiles + WAVES - 1) / WAVES;
    const int64_t most = (ncu + groups(G) - 1) / groups(G);      // about one workgroup per compute unit
    if (wpg > most) wpg = most;
    const dim3 grid((unsigned)(groups(G) * wpg));
    if (Ds % 4 == 0 && ((uintptr_t)vectors & 15) == 0)
        hipLaunchKernelGGL((encode_mfma_kernel<DP, THREADS, true>), grid, dim3(THREADS), 0, st, vectors, N, M, Ds, codewords,
                           codes, G, (int)wpg);
    else
        hipLaunchKernelGGL((encode_mfma_kernel<DP, THREADS, false>), grid, dim3(THREADS), 0, st, vectors, N, M, Ds,
                           codewords, codes, G, (int)wpg);
}

}  // namespace

extern "C" {

const char* pqkm_status_string(pqkm_status s)
{
    switch (s) {
        case PQKM_OK: return "ok";
        case PQKM_ERR_NULL: return "a required pointer is NULL";
        case PQKM_ERR_SHAPE: return "invalid shape, size, alignment or option";
        case PQKM_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case PQKM_ERR_DEVICE: return "not a gfx950 device, or a HIP call failed";
        case PQKM_ERR_TOO_LARGE: return "problem needs more scratch than the static buffer of pqkm_assign_noalloc holds";
    }
    return "unknown status";
}

size_t pqkm_workspace_bytes(int64_t N, int32_t M, int32_t K)
{
    if (!shape_ok(N, M, K)) return 0;
    return carve(N, M, K).total;
}

pqkm_status pqkm_build_tables(const float* codewords, int32_t M, int32_t Ds, float* tables, void* stream)
{
    if (!codewords || !tables) return PQKM_ERR_NULL;
    if (M < 1 || M > 64 || Ds < 1 || Ds > 12288) return PQKM_ERR_SHAPE;
    pqkm_status s = check_device();
    if (s != PQKM_OK) return s;
    hipLaunchKernelGGL(build_tables_kernel, dim3(L, M), dim3(256), (size_t)Ds * sizeof(float), (hipStream_t)stream,
                       codewords, Ds, tables);
    return launched();
}

pqkm_status pqkm_encode(const float* vectors, int64_t N, int32_t M, int32_t Ds, const float* codewords,
                        uint8_t* codes, void* stream)
{
    if (N < 0 || M < 1 || M > 64 || Ds < 1 || Ds > 12288 || N > (int64_t)0x7fffffff * 256) return PQKM_ERR_SHAPE;
    if (!codewords || (N > 0 && (!vectors || !codes))) return PQKM_ERR_NULL;
    pqkm_status s = check_device();
    if (s != PQKM_OK) return s;
    if (N == 0) return PQKM_OK;
    hipStream_t st = (hipStream_t)stream;
    if (Ds <= 4) launch_encode<4, 1024>(vectors, N, M, Ds, codewords, codes, st);
    else if (Ds <= 8) launch_encode<8, 1024>(vectors, N, M, Ds, codewords, codes, st);
    else if (Ds <= 16) launch_encode<16, 1024>(vectors, N, M, Ds, codewords, codes, st);
    else if (Ds <= 32) launch_encode<32, 1024>(vectors, N, M, Ds, codewords, codes, st);
    else if (Ds <= 64) launch_encode<64, 512>(vectors, N, M, Ds, codewords, codes, st);
    else if (Ds <= 128) launch_encode<128, 512>(vectors, N, M, Ds, codewords, codes, st);
    else
        hipLaunchKernelGGL(encode_generic_kernel, dim3((unsigned)((N + 255) / 256), (unsigned)M), dim3(256), 0, st, vectors,
                           N, M, Ds, codewords, codes);
    return launched();
}

pqkm_status pqkm_decode(const uint8_t* codes, int64_t N, int32_t M, int32_t Ds, const float* codewords,
                        float* vectors, void* stream)
{
    if (N < 0 || M < 1 || M > 64 || Ds < 1 || Ds > 12288) return PQKM_ERR_SHAPE;
    if (!codewords || (N > 0 && (!vectors || !codes))) return PQKM_ERR_NULL;
    pqkm_status s = check_device();
    if (s != PQKM_OK) return s;
    if (N == 0) return PQKM_OK;
    const int64_t total = N * M * Ds;
    if ((total + 255) / 256 > (int64_t)0x7fffffff) return PQKM_ERR_SHAPE;
    const unsigned wide = (unsigned)((total + 1024 * DECODE_PER - 1) / (1024 * DECODE_PER));
    // Lengths that are no multiple of 4: a thread fetches its four elements one after the other, which pays by the wider stores.
    // Small outputs stay in the caches and gain nothing from them, and short subvectors of many subspaces are bound by the
    // fetches.  One element per thread / four, us: M = 4, Ds = 6: 7.1 / 9.0 at N = 1e5, 53 / 37 at 1e6; M = 32, Ds = 3: 23 / 33 at
    // 1e5, 273 / 275 at 1e6; M = 32, Ds = 9: 61 / 61 at 1e5, 733 / 581 at 1e6.
    const bool single = Ds % 4 != 0 && (total < ((int64_t)1 << 22) || (M >= 16 && Ds < 8 && total < ((int64_t)1 << 26)));
    if ((((uintptr_t)vectors | (uintptr_t)codewords) & 15) != 0 || single)
        hipLaunchKernelGGL(decode_element_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                           codes, total, M, Ds, codewords, vectors);
    else if (Ds % 4 == 0)
        hipLaunchKernelGGL((decode_kernel<true>), dim3(wide), dim3(256), 0, (hipStream_t)stream, codes, total, M, Ds,
                           codewords, vectors);
    else
        hipLaunchKernelGGL((decode_kernel<false>), dim3(wide), dim3(256), 0, (hipStream_t)stream, codes, total, M, Ds,
                           codewords, vectors);
    return launched();
}

pqkm_status pqkm_assign(const uint8_t* codes, int64_t N, int32_t M, const uint8_t* centers, int32_t K,
                        const float* tables, int32_t* assign, float* dist, void* workspace, size_t workspace_bytes,
                        void* stream)
{
    if (!shape_ok(N, M, K)) return PQKM_ERR_SHAPE;
    if (!centers || !tables || (N > 0 && (!codes || !assign))) return PQKM_ERR_NULL;
    const Carve c = carve(N, M, K);
    pqkm_status s = check_workspace(workspace, workspace_bytes, c.total);
    if (s != PQKM_OK) return s;
    if ((s = check_device()) != PQKM_OK) return s;
    return assign_impl(options_snapshot(), c, codes, N, M, centers, K, tables, assign, dist, workspace,
                       (hipStream_t)stream);
}

pqkm_status pqkm_assign_noalloc(const uint8_t* codes, int64_t N, int32_t M, const uint8_t* centers, int32_t K,
                                const float* tables, int32_t* assign, float* dist, void* stream)
{
    if (!shape_ok(N, M, K)) return PQKM_ERR_SHAPE;
    if (!centers || !tables || (N > 0 && (!codes || !assign))) return PQKM_ERR_NULL;
    const Carve c = carve(N, M, K);
    if (c.total > (size_t)PQKM_NOALLOC_SCRATCH_BYTES) return PQKM_ERR_TOO_LARGE;
    pqkm_status s = check_device();
    if (s != PQKM_OK) return s;
    void* ws = nullptr;
    if ((s = scratch_of_current_device(&ws)) != PQKM_OK) return s;
    Options opt = options_snapshot();
    opt.profile = 0;                        // the event pairs of the profile option are created on demand
    return assign_impl(opt, c, codes, N, M, centers, K, tables, assign, dist, ws, (hipStream_t)stream);
}

size_t pqkm_index_workspace_bytes(int32_t M, int32_t K)
{
    if (M < 2 || M > 64 || K < 1) return 0;
    return index_carve(M, K).total;
}

pqkm_status pqkm_assign_indexed(const uint8_t* codes, int64_t N, int32_t M, const uint8_t* centers, int32_t K,
                                const float* tables, int32_t* assign, float* dist, void* workspace,
                                size_t workspace_bytes, void* stream)
{
    if (!shape_ok(N, M, K) || M < 2 || N > (int64_t)0x7fffffff * 256) return PQKM_ERR_SHAPE;
    if (!centers || !tables || (N > 0 && (!codes || !assign))) return PQKM_ERR_NULL;
    const IndexCarve c = index_carve(M, K);
    pqkm_status s = check_workspace(workspace, workspace_bytes, c.total);
    if (s != PQKM_OK) return s;
    if ((s = check_device()) != PQKM_OK) return s;
    return assign_indexed_impl(c, codes, N, M, centers, K, tables, assign, dist, static_cast<char*>(workspace),
                               (hipStream_t)stream);
}

size_t pqkm_check_workspace_bytes(int64_t n_sample, int32_t M, int32_t K)
{
    if (!shape_ok(n_sample, M, K) || M < 2) return 0;
    const size_t a = carve(n_sample, M, K).total, b = index_carve(M, K).total;
    return (a > b ? a : b) + align256((size_t)n_sample * sizeof(int32_t));
}

pqkm_status pqkm_check(const uint8_t* sample_codes, int64_t n_sample, int32_t M, const uint8_t* centers, int32_t K,
                       const float* tables, int32_t trials, void* workspace, size_t workspace_bytes, void* stream,
                       int32_t* use_index, float* scan_ms, float* index_ms)
{
    if (!shape_ok(n_sample, M, K) || M < 2 || n_sample < 1 || trials < 1) return PQKM_ERR_SHAPE;
    if (!centers || !tables || !sample_codes || !use_index) return PQKM_ERR_NULL;
    const Carve ca = carve(n_sample, M, K);
    const IndexCarve ci = index_carve(M, K);
    const size_t shared = ca.total > ci.total ? ca.total : ci.total;
    pqkm_status s = check_workspace(workspace, workspace_bytes, shared + align256((size_t)n_sample * sizeof(int32_t)));
    if (s != PQKM_OK) return s;
    if ((s = check_device()) != PQKM_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    char* ws = static_cast<char*>(workspace);
    int32_t* out = reinterpret_cast<int32_t*>(ws + shared);
    Options opt = options_snapshot();
    opt.profile = 0;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return PQKM_ERR_DEVICE;
    if (hipEventCreate(&e1) != hipSuccess) { hipEventDestroy(e0); return PQKM_ERR_DEVICE; }
    float best_ms[2] = {0.f, 0.f};
    for (int which = 0; which < 2 && s == PQKM_OK; ++which) {
        for (int t = 0; t <= trials && s == PQKM_OK; ++t) {          // trial 0 is a warm-up and is not counted
            if (hipEventRecord(e0, st) != hipSuccess) { s = PQKM_ERR_DEVICE; break; }
            s = which == 0 ? assign_impl(opt, ca, sample_codes, n_sample, M, centers, K, tables, out, nullptr, ws, st)
                           : assign_indexed_impl(ci, sample_codes, n_sample, M, centers, K, tables, out, nullptr, ws, st);
            if (s != PQKM_OK) break;
            float ms = 0.f;
            if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { s = PQKM_ERR_DEVICE; break; }
            if (t == 1 || (t > 1 && ms < best_ms[which])) best_ms[which] = ms;
        }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (s != PQKM_OK) return s;
    if (scan_ms) *scan_ms = best_ms[0];
    if (index_ms) *index_ms = best_ms[1];
    *use_index = best_ms[1] < best_ms[0] ? 1 : 0;
    return PQKM_OK;
}

pqkm_status pqkm_update(const uint8_t* codes, int64_t N, int32_t M, const int32_t* assign, int32_t K,
                        const float* tables, uint8_t* centers, uint32_t* hist, uint32_t* counts, void* workspace,
                        size_t workspace_bytes, void* stream)
{
    if (!shape_ok(N, M, K)) return PQKM_ERR_SHAPE;
    if (!centers || !tables || (N > 0 && (!codes || !assign))) return PQKM_ERR_NULL;
    const Carve c = carve(N, M, K);
    pqkm_status s = check_workspace(workspace, workspace_bytes, c.total);
    if (s != PQKM_OK) return s;
    if ((s = check_device()) != PQKM_OK) return s;
    return update_impl(options_snapshot(), c, codes, N, M, assign, K, tables, centers, hist, counts, workspace,
                       (hipStream_t)stream);
}

pqkm_status pqkm_update_naive(const uint8_t* codes, int64_t N, int32_t M, const int32_t* assign, int32_t K,
                              const float* tables, uint8_t* centers, double* cost, void* workspace,
                              size_t workspace_bytes, void* stream)
{
    if (!shape_ok(N, M, K) || N > (int64_t)0xffffffff) return PQKM_ERR_SHAPE;
    if (!centers || !tables || (N > 0 && (!codes || !assign))) return PQKM_ERR_NULL;
    const Carve c = carve(N, M, K);
    pqkm_status s = check_workspace(workspace, workspace_bytes, c.total);
    if (s != PQKM_OK) return s;
    if ((s = check_device()) != PQKM_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    uint32_t *start, *sidx;
    sort_by_cluster(assign, N, K, c, static_cast<char*>(workspace), &start, &sidx, st);
    // grid (K, M): K up to 2^31 - 1 fits the x dimension
    hipLaunchKernelGGL(naive_update_kernel, dim3((unsigned)K, (unsigned)M), dim3(256), 0, st, codes, M, start, sidx,
                       tables, centers, cost);
    return launched();
}

pqkm_status pqkm_fit(const uint8_t* codes, int64_t N, int32_t M, const float* tables, int32_t K, uint8_t* centers,
                     int32_t iters, int32_t* assign, uint32_t* hist, uint32_t* counts, void* workspace,
                     size_t workspace_bytes, void* stream)
{
    if (!shape_ok(N, M, K) || iters < 0) return PQKM_ERR_SHAPE;
    if (!centers || !tables || (N > 0 && (!codes || !assign))) return PQKM_ERR_NULL;
    const Carve c = carve(N, M, K);
    pqkm_status s = check_workspace(workspace, workspace_bytes, c.total);
    if (s != PQKM_OK) return s;
    if ((s = check_device()) != PQKM_OK) return s;
    const Options opt = options_snapshot();
    Carried carried;                        // the codes do not change between iterations: they are regrouped once
    for (int it = 0; it < iters; ++it) {
        BucketLink link = bucket_request(opt, N, M, K);
        s = assign_impl(opt, c, codes, N, M, centers, K, tables, assign, nullptr, workspace, (hipStream_t)stream, &carried,
                        &link);
        if (s != PQKM_OK) return s;
        s = update_impl(opt, c, codes, N, M, assign, K, tables, centers, hist, counts, workspace, (hipStream_t)stream,
                        &link);
        if (s != PQKM_OK) return s;
    }
    return PQKM_OK;
}

// extra workspace of pqkm_fit_until, placed after the pqkm_fit carve
struct UntilCarve { size_t prev_off, dist_off, pa_off, ph_off, out_off, total; };

static UntilCarve until_carve(int64_t N, int M, int K)
{
    UntilCarve u{};
    size_t off = carve(N, M, K).total;
    u.prev_off = off;  off += align256((size_t)N * sizeof(int32_t));
    u.dist_off = off;  off += align256((size_t)N * sizeof(float));
    u.pa_off = off;    off += align256((size_t)STAT_BLOCKS * sizeof(StatPartial));
    u.ph_off = off;    off += align256((size_t)STAT_BLOCKS * sizeof(StatPartial));
    u.out_off = off;   off += 256;
    u.total = off;
    return u;
}

size_t pqkm_fit_until_workspace_bytes(int64_t N, int32_t M, int32_t K)
{
    if (!shape_ok(N, M, K)) return 0;
    return until_carve(N, M, K).total;
}

pqkm_status pqkm_fit_until(const uint8_t* codes, int64_t N, int32_t M, const float* tables, int32_t K,
                           uint8_t* centers, int32_t max_iters, int32_t* assign, uint32_t* hist, uint32_t* counts,
                           pqkm_iter_stats* stats, int32_t* iters_done, void* workspace, size_t workspace_bytes,
                           void* stream)
{
    if (!shape_ok(N, M, K) || max_iters < 0) return PQKM_ERR_SHAPE;
    if (!centers || !tables || (N > 0 && (!codes || !assign))) return PQKM_ERR_NULL;
    const UntilCarve u = until_carve(N, M, K);
    pqkm_status s = check_workspace(workspace, workspace_bytes, u.total);
    if (s != PQKM_OK) return s;
    if ((s = check_device()) != PQKM_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    char* ws = static_cast<char*>(workspace);
    const Carve c = carve(N, M, K);
    int32_t* prev = reinterpret_cast<int32_t*>(ws + u.prev_off);
    float* dist = reinterpret_cast<float*>(ws + u.dist_off);
    StatPartial* pa = reinterpret_cast<StatPartial*>(ws + u.pa_off);
    StatPartial* ph = reinterpret_cast<StatPartial*>(ws + u.ph_off);
    unsigned long long* out = reinterpret_cast<unsigned long long*>(ws + u.out_off);
    if (!hist) hist = reinterpret_cast<uint32_t*>(ws + c.hist_off);
    if (!counts) counts = reinterpret_cast<uint32_t*>(ws + c.counts_off);
    if (iters_done) *iters_done = 0;
    if (N > 0) {
        unsigned fb = (unsigned)((N + 255) / 256 < 65536 ? (N + 255) / 256 : 65536);
        hipLaunchKernelGGL(fill_i32_kernel, dim3(fb), dim3(256), 0, st, prev, N, (int32_t)-1);
    }
    const Options opt = options_snapshot();
    Carried carried;
    for (int it = 0; it < max_iters; ++it) {
        BucketLink link = bucket_request(opt, N, M, K);
        s = assign_impl(opt, c, codes, N, M, centers, K, tables, assign, dist, workspace, st, &carried, &link);
        if (s != PQKM_OK) return s;
        hipLaunchKernelGGL(iter_assign_stats_kernel, dim3(STAT_BLOCKS), dim3(256), 0, st, assign, prev, dist, N, pa);
        s = update_impl(opt, c, codes, N, M, assign, K, tables, centers, hist, counts, workspace, st, &link);
        if (s != PQKM_OK) return s;
        hipLaunchKernelGGL(iter_hist_stats_kernel, dim3(STAT_BLOCKS), dim3(256), 0, st, hist, (int64_t)K * M * L,
                           counts, K, ph);
        hipLaunchKernelGGL(iter_stats_final_kernel, dim3(1), dim3(1024), 0, st, pa, ph, out);
        unsigned long long h[4];
        if (hipMemcpyAsync(h, out, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess) return PQKM_ERR_DEVICE;
        if (hipStreamSynchronize(st) != hipSuccess) return PQKM_ERR_DEVICE;
        if (stats) {
            double d;
            memcpy(&d, &h[0], sizeof(d));
            stats[it].objective = d;
            stats[it].changed = (int64_t)h[1];
            stats[it].nonzero_bins = (int64_t)h[2];
            stats[it].nonempty = (int64_t)h[3];
        }
        if (iters_done) *iters_done = it + 1;
        if (h[1] == 0) break;
    }
    return PQKM_OK;
}

pqkm_status pqkm_set_option(const char* name, int32_t value)
{
    if (!name) return PQKM_ERR_NULL;
    std::lock_guard<std::mutex> lk(g_mu);
    if (strcmp(name, "assign_kernel") == 0) {
        if (value < 0 || value > 2) return PQKM_ERR_SHAPE;
        g_opt.assign_kernel = value;
    } else if (strcmp(name, "scan_variant") == 0) {
        if (value < 0 || value > 99) return PQKM_ERR_SHAPE;
        g_opt.scan_variant = value;
    } else if (strcmp(name, "hist_kernel") == 0) {
        if (value < 0 || value > 3) return PQKM_ERR_SHAPE;
        g_opt.hist_kernel = value;
    } else if (strcmp(name, "profile") == 0) {
        if (value < 0 || value > 3) return PQKM_ERR_SHAPE;
        g_opt.profile = value;
    } else if (strcmp(name, "scan_rounds_per_launch") == 0) {
        if (value < 0 || value > 1024) return PQKM_ERR_SHAPE;
        g_opt.rounds_per_launch = value;
    } else if (strcmp(name, "launch_codes_log2") == 0) {
        if (value < 10 || value > 40) return PQKM_ERR_SHAPE;
        g_opt.launch_codes = (int64_t)1 << value;
    } else {
        return PQKM_ERR_SHAPE;
    }
    return PQKM_OK;
}

pqkm_status pqkm_scan_plan(int64_t N, int32_t M, int32_t K, int32_t iteration, int64_t out[6])
{
    if (!out) return PQKM_ERR_NULL;
    if (!shape_ok(N, M, K) || iteration < 0) return PQKM_ERR_SHAPE;
    const Options opt = options_snapshot();
    for (int i = 0; i < 6; ++i) out[i] = 0;
    if (!tiled_scan(opt, N, M, K, nullptr, nullptr)) return PQKM_OK;
    const Carve c = carve(N, M, K);
    const BucketLink link = bucket_request(opt, N, M, K);
    const bool files_records = M == 4 && link.wanted && N <= GROUP_CHUNK_MAX - 16384 && c.bseg_off != c.pool_off;
    Carried carried;
    ScanPlan p{};
    for (int it = 0; it <= iteration; ++it) {
        p = scan_plan(M, opt, N, K, nullptr, nullptr, files_records, false, c, carried);
        carried = p.leaves;
    }
    out[0] = p.filter || p.wide ? 2 : 1;
    out[1] = p.variant;
    out[2] = p.per_launch;
    out[3] = p.lanes;
    out[4] = p.reuse ? 1 : 0;
    out[5] = p.seeded;
    return PQKM_OK;
}

pqkm_status pqkm_call_plan(int64_t N, int32_t M, int32_t K, int32_t flags, int64_t out[8])
{
    if (!out) return PQKM_ERR_NULL;
    if (!shape_ok(N, M, K) || flags < 0 || flags > 7) return PQKM_ERR_SHAPE;
    const Options opt = options_snapshot();
    const Carve c = carve(N, M, K);
    const uint8_t* codes = reinterpret_cast<const uint8_t*>((uintptr_t)(flags & 1));          // an address that is looked at only
    const uint8_t* centers = reinterpret_cast<const uint8_t*>((uintptr_t)(flags >> 1 & 1));
    for (int i = 0; i < 8; ++i) out[i] = 0;
    if (tiled_scan(opt, N, M, K, codes, centers)) {
        Carried none;
        none.alone = true;
        const ScanPlan p = scan_plan(M, opt, N, K, codes, centers, false, (flags & 4) != 0, c, none);
        out[0] = p.filter || p.wide ? 2 : 1;
        out[1] = p.variant;
        out[2] = p.dot;
    } else {
        out[2] = dot_before_rows(M, opt, N, K, codes, centers, c);
        const GatherPlan p = gather_plan(N, M, K, (((uintptr_t)codes | (uintptr_t)centers) & 3) == 0, tiled_M(M) ? c.img_bytes : 0, out[2] != 0);
        out[1] = p.per_code ? 2 : p.rows ? 1 : 0;
        out[3] = p.codes;
        out[4] = p.parts;
    }
    const HistPath path = hist_path(N, M, K, c, opt.hist_kernel, false, false);
    const UpdateRoute route = update_route(path, opt.hist_kernel, N, M, K, codes);
    out[5] = route == UPDATE_IN_VOTE_FEW ? 5 : route == UPDATE_IN_VOTE ? 6 : (int64_t)path;
    out[6] = route != UPDATE_PASS ? 1 : path == HIST_SUBSPACE ? subspace_hist(N, M, K, c).S : path == HIST_OWNER ? hist_plan(N, M, K).S : 1;
    out[7] = route == UPDATE_IN_VOTE_FEW || (route == UPDATE_PASS && (path == HIST_SUBSPACE || vote_few(N, M, K))) ? 1 : 0;
    return PQKM_OK;
}

pqkm_status pqkm_dot_scan(int64_t N, int32_t M, int32_t K, const void* workspace, int32_t out[2])
{
    if (!out) return PQKM_ERR_NULL;
    if (!shape_ok(N, M, K)) return PQKM_ERR_SHAPE;
    const Options opt = options_snapshot();
    out[0] = 0;
    out[1] = -1;
    if (!tiled_scan(opt, N, M, K, nullptr, nullptr)) return PQKM_OK;
    const Carve c = carve(N, M, K);
    const BucketLink link = bucket_request(opt, N, M, K);
    const bool files_records = M == 4 && link.wanted && N <= GROUP_CHUNK_MAX - 16384 && c.bseg_off != c.pool_off;
    out[0] = scan_plan(M, opt, N, K, nullptr, nullptr, files_records, false, c, Carried{}).dot ? 1 : 0;
    if (!workspace || !out[0]) return PQKM_OK;
    uint32_t left = 0;
    if (hipDeviceSynchronize() != hipSuccess ||
        hipMemcpy(&left, static_cast<const char*>(workspace) + c.dot_off + offsetof(DotState, left), sizeof(left), hipMemcpyDeviceToHost) != hipSuccess)
        return PQKM_ERR_DEVICE;
    out[1] = left ? 1 : 0;
    return PQKM_OK;
}

pqkm_status pqkm_profile_read(double* total_ms, int64_t* launches)
{
    return log_read(g_scan_log, total_ms, launches);
}

pqkm_status pqkm_profile_read_steps(double* total_ms, int64_t* steps)
{
    return log_read(g_step_log, total_ms, steps);
}

}  // extern "C"
