// rv.hip -- gfx950 kernels and host entry points of the per-cluster RANSAC
// velocity and heading estimator declared in include/rv.h.
//
// A single-frame call enqueues three kernels on the caller's stream:
//   prep    one thread per point: FP64 sincos of the azimuth; stages float32
//           (cos, sin) and v_d for scoring and the float32 low parts of the
//           FP64 (cos, sin) for the solves and the refit;
//           clears the optional frame-wide inlier bitmask and the per-cluster
//           best keys.  Its first workgroup plans the dispatch order: clusters
//           by decreasing size.
//   score   the hot loop.  Workgroup = (cluster, up to 1024 hypotheses).  Each
//           thread draws Philox4x32-10 seed pairs and solves the 2x2 systems in FP64
//           (Sec. 3.1, Alg. 1: seeds, slope and intercept, as the velocity profile
//           of Sec. 3.2, Eq. 6); the float32 (vx, vy) go to LDS.  By the cluster's
//           size:
//           small (score_small): the points in LDS, a thread holds up to four
//           hypotheses and counts their inliers point by point (Alg. 1's distance
//           test, two float32 FMAs, and a clamped FMA as the compare);
//           larger (score_pruned): a table of the points under a good hypothesis
//           bounds every other one's count, and only those that can still win are
//           counted, lanes = points, with a ballot and a scalar popcount;
//           calls that ask for every hypothesis's count, and tau beyond the bound's
//           range, take lanes = points for all (score_block).
//           The best (count, lowest index) key is merged per cluster with a 64-bit
//           atomic maximum (Sec. 3.1: the trial with the most inliers is kept).
//   refit   one wave per cluster, or a whole workgroup for large ones (in dense
//           frames the scoring workgroup itself): FP64 re-classification under the
//           kept hypothesis, FP64 normal-equation sums in a fixed reduction tree,
//           2x2 solve (Sec. 3.2, Eq. 7, Alg. 2) and atan2 heading (Eq. 8).
// Small frames without an inlier mask take one launch (cluster_kernel)
// that runs the same three steps per cluster in one workgroup.  A part of a
// frame (its clusters drawing with their whole-frame indexes, its points found
// through the frame's offsets minus a point base) runs the same kernels; a
// frame in host memory can be copied and estimated part by part.  The batched
// form stages, orders and describes the clusters of many frames, scores them
// from per-XCD work queues in one persistent launch (optionally in the FP16
// residual form) and refits them in one more launch.  Long clusters take
// workgroups of 1024 threads in both forms.
//
// No floating-point atomics and fixed reduction orders: results are bitwise
// reproducible run to run and independent of the other clusters in the frame.

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <vector>

#include "rv.h"
#include "rv_device.h"
#include "rv_internal.h"

// v_writelane_b32: write a wave-uniform value into one lane of a VGPR (the
// LLVM intrinsic; clang exposes no builtin for it).
__device__ int amdgcn_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

// Error text shared by every translation unit of the library.
namespace rv_internal {
thread_local char g_error[512] = "";

int fail(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_error, sizeof g_error, fmt, ap);
    va_end(ap);
    return code;
}

// Stage timing (rv_stage_timing / rv_stage_times): events recorded around the
// kernels of a call.
std::mutex g_timing_mutex;
bool g_timing = false;
std::vector<TimedCall> g_pending;   // recorded, not yet read
std::vector<TimedCall> g_free;      // reusable event sets

bool take_timed_call(TimedCall &tc) {
    std::lock_guard<std::mutex> lock(g_timing_mutex);
    if (!g_timing) return false;
    if (!g_free.empty()) {
        tc = g_free.back();
        g_free.pop_back();
        return true;
    }
    for (int i = 0; i <= kStages; ++i)
        if (hipEventCreate(&tc.ev[i]) != hipSuccess) return false;
    return true;
}

void keep_timed_call(const TimedCall &tc) {
    std::lock_guard<std::mutex> lock(g_timing_mutex);
    g_pending.push_back(tc);
}
}  // namespace rv_internal

namespace {

constexpr int kScoreBlock = 256;        // score: 4 waves x 64 hypotheses, one per thread
constexpr int kRefitBlock = 256;
constexpr int kLongBlock = 1024;        // score and refit of long clusters (long_clusters)
// Clusters from this size on are refit by a whole workgroup, smaller ones by a wave
// each, with the same bits (see refit_cluster).  Many clusters (more than fit the chip
// at eight workgroups per CU): from 1024 points, a wave alone being the cheaper form
// until its chain is the longest thing left.  Fewer: from 256 points, where only the chain
// counts (refit of 700 clusters of 8 to 1024 points 10.8 us from 1024 on, 8.1 us from 256
// on; of 300 clusters of 512 points 9.8 and 8.2, of 1000 of 256 points 8.8 and 8.7).
constexpr int kRefitManyClusters = 2048;
constexpr int kRefitBigPoints = 1024;
constexpr int kRefitBigClass = 41;     // size class of 1024 points
constexpr int kRefitBigClassFew = 33;  // and of 256 points

__host__ __device__ constexpr int refit_big_class(int64_t n_clusters) {
    return n_clusters >= kRefitManyClusters ? kRefitBigClass : kRefitBigClassFew;
}
constexpr int kXcds = 8;                // MI355X: 8 XCDs, workgroups dealt round-robin
// Where a scoring workgroup has all hypotheses of a cluster (1024 in four blocks, see
// score_rounds), clusters from this size on are split between two: the largest
// workgroup sets the end of a frame whose workgroups are few more than fit the chip.
// Scoring and refit of 4096 clusters of 8 to 4096 points at 20, 60 and 90 % outliers 81,
// 182 and 312 us unsplit, 81, 137 and 234 us split; 2100 of 16 to 8192 points 110, 290
// and 560 us, 79, 227 and 292 us; but 2100 of 2048 points each 100 and 104 us at 20 %.
constexpr int64_t kSplitPoints = 2048;
constexpr int kSplitClass = 45;         // size class of kSplitPoints
constexpr int32_t kSplitParts = 2;

// The most clusters that are split (the grid has room for them), a multiple of kXcds.
// More than n_points / kSplitPoints can be that large where offsets are not ascending.
__host__ __device__ constexpr int64_t split_max(int64_t n_clusters, int64_t n_points) {
    const int64_t room = n_points / kSplitPoints < n_clusters ? n_points / kSplitPoints : n_clusters;
    return (room + kXcds - 1) / kXcds * kXcds;
}
constexpr int kPrepBlock = 256;
constexpr int kRowsMax = 16;            // register rows per pass, the most a tuning may name
constexpr int kPassRows = 12;           // register rows per pass, the most the float32 loop holds
// And in score_kernel, which with twelve spills (a wave that uses scratch starts later): full
// count of 4096 clusters of 256 points 35.9 and 33.7 us, of 64 of 65,536 points 1110 and
// 1135 us a call.  (cluster_kernel spills either way: 10.3 us with twelve, 10.5 with ten.)
constexpr int kFrameRows = 10;
constexpr int kHypGroup = 4;            // hypotheses per LDS fetch in the scoring loop
constexpr int kSizeClasses = 128;       // quarter-octave size classes for the dispatch order
constexpr int64_t kPlanMaxClusters = 1 << 16;  // above this, clusters run in index order
// ---------------------------------------------------------------------------
// Device helpers
// ---------------------------------------------------------------------------

// One staged point: float32 (cos, sin) and v_d for scoring (v_d = +inf marks a
// point whose azimuth or Doppler value is not finite), and beside them, in an array
// of their own, the float32 low parts of the FP64 (cos, sin) for the solves and the
// refit (cs64() below).  The sweeps over a cluster's points read the 12-byte records
// only, and of large clusters they miss L2 (2048 resident workgroups); the seeds'
// gathers and the refit read both.  In one 20-byte record a seed is fewer cache lines,
// but every sweep reads all of it: 256 frames 2357 us, split 2251 us; the dense frame
// 92.9 and 88.8 us (scoring 257 MB a launch from beyond L2 with the record); clusters
// of 64 points, all gathers, 276 and 284 us.
struct StagedPoint {
    float c, s, v;
};
struct StagedLow {
    float c, s;
};
static_assert(sizeof(StagedPoint) == 12 && sizeof(StagedLow) == 8, "packed");

// Where points are staged.
struct Staging {
    StagedPoint *points;
    StagedLow *low;
};

// A frame's staged points and the caller's azimuths (for the seed-separation
// test).
struct Points {
    const StagedPoint *staged;
    const StagedLow *low;
    const float *theta;
};

// FP64 (cos, sin) of a staged point: the float32 value plus its float32 low
// part, c = hi + lo (an exact FP64 sum), within 2^-49 of the FP64 sincos.
// Staging 8 bytes per point for the low parts instead of 16 for the FP64 pair
// shortens the staging kernel, which is bound by its bytes.
__device__ __forceinline__ double2 cs64(const StagedPoint &p, const StagedLow &low) {
    return make_double2((double)p.c + (double)low.c, (double)p.s + (double)low.s);
}

struct Hypothesis {
    double vx, vy;
    bool valid;
};

// The two seed points of a hypothesis.
struct Seeds {
    int64_t pi, pj;
    StagedPoint a, b;
    StagedLow al, bl;
};

// Seed pair of hypothesis h of cluster k.  No branch: all loads are in flight
// together.
__device__ __forceinline__ Seeds draw_seeds(const Points &pts, Span sp, uint32_t h, uint32_t k,
                                            uint32_t key0, uint32_t key1) {
    const uint4 u = philox4x32_10(make_uint4(h, k, 0u, 0u), key0, key1);
    uint32_t i, j;
    seed_pair(u.x, u.y, (uint32_t)sp.n, i, j);
    Seeds d;
    d.pi = sp.lo + i;
    d.pj = sp.lo + j;
    d.a = pts.staged[d.pi];
    d.b = pts.staged[d.pj];
    d.al = pts.low[d.pi];
    d.bl = pts.low[d.pj];
    return d;
}

// Validity and the FP64 2x2 solve of v_d = vx cos + vy sin at the two seeds
// (Cramer's rule); an invalid pair's solve (possibly inf or NaN) is replaced by
// NaN.
__device__ __forceinline__ Hypothesis solve_seeds(const Points &pts, const Seeds &d) {
    const double2 ai = cs64(d.a, d.al), bj = cs64(d.b, d.bl);
    const double ci = ai.x, si = ai.y, cj = bj.x, sj = bj.y;
    const double dvi = d.a.v, dvj = d.b.v;
    const double det = ci * sj - si * cj;
    Hypothesis hy;
    hy.valid = ((int)isfinite(d.a.v) & (int)isfinite(d.b.v)) != 0;
    // The determinant is sin(theta_j - theta_i) within 2^-46, and |sin x| <=
    // |x|: above the separation limit (with room for that error) the pair is
    // separated.  Only below it are the azimuths themselves read.
    if (!(fabs(det) > 1.0005 * RV_MIN_SEED_SEPARATION) && hy.valid)
        hy.valid = fabs((double)pts.theta[d.pj] - (double)pts.theta[d.pi]) >= RV_MIN_SEED_SEPARATION;
    const double inv_det = 1.0 / det;
    const double vx = (dvi * sj - dvj * si) * inv_det;
    const double vy = (ci * dvj - cj * dvi) * inv_det;
    hy.vx = hy.valid ? vx : __builtin_nan("");
    hy.vy = hy.valid ? vy : __builtin_nan("");
    return hy;
}

// Hypothesis h of cluster k.
__device__ __forceinline__ Hypothesis make_hypothesis(const Points &pts, Span sp, uint32_t h,
                                                      uint32_t k, uint32_t key0, uint32_t key1) {
    return solve_seeds(pts, draw_seeds(pts, sp, h, k, key0, key1));
}

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------

// Size class of a cluster for the dispatch order: quarter-octave buckets of n,
// larger n -> larger class; clusters with fewer than two points get class 0.
__device__ __forceinline__ int size_class(int64_t n) {
    if (n < 2) return 0;
    const uint32_t u = n > 0x7FFFFFFF ? 0x7FFFFFFFu : (uint32_t)n;
    const int e = 31 - __builtin_clz(u);                      // floor(log2 n) >= 1
    const int frac = e >= 2 ? (int)((u >> (e - 2)) & 3u) : (int)((u << (2 - e)) & 3u);
    const int c = 1 + 4 * e + frac;
    return c < kSizeClasses ? c : kSizeClasses - 1;
}

// Dispatch order of the clusters: a counting sort by decreasing size class, so
// the longest workgroups start first (longest-processing-time-first).  The
// order inside a class depends on atomics; it only affects scheduling.
// Each thread takes clusters tid, tid + 256, ... in groups of kPlanUnroll, whose
// offsets are all loaded before any of their LDS atomics; the exclusive scan
// over the classes (largest first) is one wave's prefix sum, two classes per
// lane.  This workgroup runs beside the staging workgroups and sets the prep
// kernel's length when it is the slower one.
static_assert(kSizeClasses == 2 * kWave, "the class scan takes two classes per lane");

// Exclusive prefix sum of x over the lanes of one full wave.
__device__ __forceinline__ uint32_t wave_exclusive_sum(uint32_t x, int lane) {
    uint32_t incl = x;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += y;
    }
    return incl - x;
}

// Start of each size class in the dispatch order (largest class first), the
// number of clusters refit by a whole workgroup (n_big[0]) and split between scoring
// workgroups (n_big[1]); the first wave of the block.
__device__ __forceinline__ void plan_scan(const uint32_t *count, uint32_t *start, int big_class,
                                          int64_t most_split, int64_t *__restrict__ n_big) {
    if (threadIdx.x < kWave) {
        // Position q = 0, 1, ... in the dispatch order is class kSizeClasses - 1 - q.
        const int lane = threadIdx.x;
        const int c_hi = kSizeClasses - 1 - 2 * lane, c_lo = c_hi - 1;
        const uint32_t a = count[c_hi], b = count[c_lo];
        const uint32_t excl = wave_exclusive_sum(a + b, lane);
        start[c_hi] = excl;
        start[c_lo] = excl + a;
        // Clusters refit by a whole workgroup: classes big_class and up; clusters split
        // between scoring workgroups, a multiple of kXcds.
        if (c_hi == big_class) n_big[0] = excl + a;
        if (c_lo == big_class) n_big[0] = excl + a + b;
        if (c_hi == kSplitClass || c_lo == kSplitClass) {
            const int64_t n = excl + a + (c_lo == kSplitClass ? b : 0u);
            const int64_t whole = (n + kXcds - 1) / kXcds * kXcds;
            n_big[1] = whole < most_split ? whole : most_split;
        }
    }
}

constexpr int kPlanUnroll = 16;
__device__ void plan_order(const int32_t *__restrict__ off, int64_t point_base, int64_t n_clusters,
                           int64_t n_points, int big_class, int32_t *__restrict__ order,
                           int64_t *__restrict__ n_big) {
    __shared__ uint32_t count[kSizeClasses];
    __shared__ uint32_t start[kSizeClasses];
    for (int c = threadIdx.x; c < kSizeClasses; c += kPrepBlock) count[c] = 0;
    __syncthreads();
    const int64_t group = (int64_t)kPlanUnroll * kPrepBlock;
    if (n_clusters <= group) {
        // One group: every thread's classes stay in registers from the count
        // to the placement, so the offsets are read once (their loads queue
        // behind the staging traffic of the other workgroups).
        int cls[kPlanUnroll];
#pragma unroll
        for (int u = 0; u < kPlanUnroll; ++u) {
            const int64_t k = threadIdx.x + (int64_t)u * kPrepBlock;
            cls[u] = k < n_clusters ? size_class(cluster_span(off, k, n_points, point_base).n) : -1;
        }
#pragma unroll
        for (int u = 0; u < kPlanUnroll; ++u)
            if (cls[u] >= 0) atomicAdd(&count[cls[u]], 1u);
        __syncthreads();
        plan_scan(count, start, big_class, split_max(n_clusters, n_points), n_big);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPlanUnroll; ++u) {
            if (cls[u] >= 0) {
                const uint32_t pos = atomicAdd(&start[cls[u]], 1u);
                order[pos] = (int32_t)(threadIdx.x + u * kPrepBlock);
            }
        }
        return;
    }
    for (int64_t k0 = threadIdx.x; k0 < n_clusters; k0 += group) {
        int cls[kPlanUnroll];
#pragma unroll
        for (int u = 0; u < kPlanUnroll; ++u) {
            const int64_t k = k0 + (int64_t)u * kPrepBlock;
            cls[u] = k < n_clusters ? size_class(cluster_span(off, k, n_points, point_base).n) : -1;
        }
#pragma unroll
        for (int u = 0; u < kPlanUnroll; ++u)
            if (cls[u] >= 0) atomicAdd(&count[cls[u]], 1u);
    }
    __syncthreads();
    plan_scan(count, start, big_class, split_max(n_clusters, n_points), n_big);
    __syncthreads();
    for (int64_t k0 = threadIdx.x; k0 < n_clusters; k0 += group) {
        int cls[kPlanUnroll];
#pragma unroll
        for (int u = 0; u < kPlanUnroll; ++u) {
            const int64_t k = k0 + (int64_t)u * kPrepBlock;
            cls[u] = k < n_clusters ? size_class(cluster_span(off, k, n_points, point_base).n) : -1;
        }
#pragma unroll
        for (int u = 0; u < kPlanUnroll; ++u) {
            if (cls[u] >= 0) {
                const uint32_t pos = atomicAdd(&start[cls[u]], 1u);
                order[pos] = (int32_t)(k0 + (int64_t)u * kPrepBlock);
            }
        }
    }
}

// Stages point p: FP64 sincos of its azimuth, float32 (cos, sin) and v_d for
// scoring, and the float32 low parts of the FP64 (cos, sin) (c - (double)(float)c,
// rounded) for the solves and the refit.  A non-finite point is staged as
// (0, 0, +inf) with zero low parts: its float32 residual is inf or NaN, never
// below tau, and +inf marks it for the solves and the refit.
__device__ __forceinline__ void stage_point(const float *__restrict__ theta,
                                            const float *__restrict__ vd, int64_t p,
                                            const Staging &staged) {
    const float t = theta[p], v = vd[p];
    double s, c;
    sincos((double)t, &s, &c);
    const bool ok = isfinite(t) && isfinite(v);
    const float ch = ok ? (float)c : 0.0f, sh = ok ? (float)s : 0.0f;
    StagedPoint q;
    q.c = ch;
    q.s = sh;
    q.v = ok ? v : __builtin_inff();
    StagedLow low;
    low.c = ok ? (float)(c - (double)ch) : 0.0f;
    low.s = ok ? (float)(s - (double)sh) : 0.0f;
    staged.points[p] = q;
    staged.low[p] = low;
}

// Block 0 plans the order (when `order` is non-null); it is dispatched first,
// so the planning overlaps the staging.  Blocks [1, gridDim.x) stage the
// points and clear the per-cluster best keys.
__global__ __launch_bounds__(kPrepBlock) void prep_kernel(
    const float *__restrict__ theta, const float *__restrict__ vd, int64_t n_points,
    Staging staged, uint32_t *__restrict__ bits,
    int64_t n_words, const int32_t *__restrict__ off, int64_t point_base, int64_t n_clusters,
    int32_t big_class, int32_t *__restrict__ order, int64_t *__restrict__ n_big,
    unsigned long long *__restrict__ best_key) {
    if (blockIdx.x == 0) {
        if (order != nullptr)
            plan_order(off, point_base, n_clusters, n_points, big_class, order, n_big);
        return;
    }
    const int64_t p = (int64_t)(blockIdx.x - 1) * kPrepBlock + threadIdx.x;
    if (p < n_clusters) best_key[p] = 0;
    if (p < n_points) stage_point(theta, vd, p, staged);
    if (bits != nullptr && p < n_words) bits[p] = 0u;
}

// The point at byte offset `at` of a row (a wave-uniform base, so that the load takes
// it from scalar registers; indexing the row by the lane cost a 64-bit vector
// multiply-add for every row).
__device__ __forceinline__ const StagedPoint &row_point(const StagedPoint *row, uint32_t at) {
    return *reinterpret_cast<const StagedPoint *>(reinterpret_cast<const char *>(row) + at);
}

// R rows of 64 points per lane (registers) against ng groups of kHypGroup
// hypotheses read from LDS (broadcast reads: every lane gets the same (vx, vy));
// returns the count of hypothesis q of the wave in lane q.  kScalarLoop: the
// group count is read as a wave-uniform value, which keeps the loop counter on
// the scalar unit (measured 1 % faster in the persistent batched kernel, 0.5 %
// slower in the single-frame kernel, whose schedule it changes).
template <int R, bool kScalarLoop>
__device__ __forceinline__ uint32_t count_rows(const float (&c)[R], const float (&s)[R],
                                               const float (&v)[R], const float4 *hp, int ng,
                                               float tau) {
    uint32_t counts = 0;
    const int n_groups = kScalarLoop ? __builtin_amdgcn_readfirstlane(ng) : ng;
    for (int g = 0; g < n_groups; ++g) {
        const float4 h0 = hp[2 * g], h1 = hp[2 * g + 1];
        const float hx[kHypGroup] = {h0.x, h0.z, h1.x, h1.z};
        const float hy[kHypGroup] = {h0.y, h0.w, h1.y, h1.w};
#pragma unroll
        for (int u = 0; u < kHypGroup; ++u) {
            uint32_t n = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float t = __builtin_fmaf(-hx[u], c[r], v[r]);
                const float e = __builtin_fmaf(-hy[u], s[r], t);
                n += (uint32_t)__builtin_popcountll(
                    __builtin_amdgcn_ballot_w64(__builtin_fabsf(e) < tau));
            }
            counts = (uint32_t)amdgcn_writelane((int)n, g * kHypGroup + u, (int)counts);
            // One hypothesis at a time: interleaving several keeps R ballot masks
            // per hypothesis live and spills scalar registers.
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return counts;
}

// count_rows on the npts points from `chunk` on (the rest of the rows padded with
// a point that never counts).
template <int R, bool kScalarLoop = false>
__device__ __forceinline__ uint32_t score_rows(const StagedPoint *__restrict__ chunk, int npts,
                                               int lane, const float4 *hp, int ng, float tau) {
    float c[R], s[R], v[R];
    const uint32_t at = (uint32_t)lane * (uint32_t)sizeof(StagedPoint);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        // Uniform row base and row length, one 32-bit lane offset: no per-row address
        // arithmetic on the vector unit.
        const int len = npts - r * kWave;
        c[r] = 0.0f;
        s[r] = 0.0f;
        v[r] = __builtin_inff();
        if (lane < len) {
            const StagedPoint &q = row_point(chunk + r * kWave, at);
            c[r] = q.c;
            s[r] = q.s;
            v[r] = q.v;
        }
    }
    return count_rows<R, kScalarLoop>(c, s, v, hp, ng, tau);
}

// Inlier counts of the wave's nh hypotheses (LDS at hp) over all points of the
// cluster, rows_max (at most kMaxRows are used) register rows of points per
// pass; lane q returns the count of hypothesis q.
template <int kMaxRows = kPassRows, bool kScalarLoop = false>
__device__ __forceinline__ uint32_t score_cluster(const Points &pts, Span sp, int lane,
                                                  const float4 *hp, int nh, float tau,
                                                  int rows_max) {
    const int ng = (nh + kHypGroup - 1) / kHypGroup;
    const int64_t end = sp.lo + sp.n;
    const int64_t pass = (int64_t)(rows_max < kMaxRows ? rows_max : kMaxRows) * kWave;
    uint32_t total = 0;
    for (int64_t base = sp.lo; base < end; base += pass) {
        const int64_t left = end - base;
        const int npts = (int)(left < pass ? left : pass);
        const int rows = (npts + kWave - 1) / kWave;
        const StagedPoint *chunk = pts.staged + base;
        switch (rows) {
#define RV_ROWS(R)                                                                   \
    case R:                                                                          \
        if constexpr (R <= kMaxRows)                                                 \
            total += score_rows<R, kScalarLoop>(chunk, npts, lane, hp, ng, tau); \
        break;
            RV_ROWS(1) RV_ROWS(2) RV_ROWS(3) RV_ROWS(4) RV_ROWS(5) RV_ROWS(6) RV_ROWS(7)
            RV_ROWS(8) RV_ROWS(9) RV_ROWS(10) RV_ROWS(11) RV_ROWS(12)
#undef RV_ROWS
            default: break;
        }
    }
    return total;
}

// The last t = n mod 64 points of a cluster, when t < kTailLanesMax, are
// scored with lanes = hypotheses instead of as one partly idle row: a row
// costs two FMAs and a compare for 64 lanes whatever t is, while each tail
// point costs every lane two FMAs, a compare and an add (about 12 SIMD-cycles
// per point against about 10 per row and hypothesis), so below about 50 points
// the tail is cheaper this way (thresholds of 32, 48 and 63 measured alike:
// about 5 % off the small frame, 1 % off the batched step, no change on the
// dense frame).  Thread tid holds hypothesis tid of the block
// in both forms, so the two partial counts add up in the same thread; the
// residual and the test are the rows form's, so every count is the same bit
// for bit.
constexpr int kTailLanesMax = 32;


// Points held in LDS for scoring with lanes = hypotheses: a cluster's tail, a
// whole small cluster, or a sample.
constexpr int kLaneTile = 256;  // the largest cluster scored whole this way
template <int N>
struct LaneTile {
    float4 c[N / 4], s[N / 4], v[N / 4];  // padded with (0, 0, +inf)
};

__device__ __forceinline__ int lanes_tail(int64_t n) {
    const int t = (int)(n % kWave);
    return t < kTailLanesMax ? t : 0;
}

// One staged point held by a thread between its loads and its LDS store, so
// that the loads can be issued before other long-latency work (a hypothesis's
// seed loads) and stored after it.
struct PointLoad {
    float c, s, v;
};

// Thread tid's point among the `count` points from `first` (a valid point of
// the span for the other threads: every load is in bounds, none is used).
__device__ __forceinline__ PointLoad load_point(const Points &pts, int64_t first, int count) {
    const int tid = threadIdx.x;
    const int64_t p = first + (tid < count ? tid : 0);
    const StagedPoint &q = pts.staged[p];
    PointLoad L;
    L.c = q.c;
    L.s = q.s;
    L.v = q.v;
    return L;
}

// Point p of a cluster's n (its last one past the end: in bounds, not used).
__device__ __forceinline__ PointLoad load_at(const StagedPoint *points, uint32_t p, uint32_t n) {
    const StagedPoint &q = points[p < n ? p : n - 1];
    PointLoad L;
    L.c = q.c;
    L.s = q.s;
    L.v = q.v;
    return L;
}

// Stores the points of load_point into LDS as float4 quads, padded to a
// multiple of four with (0, 0, +inf), a point that never counts; the caller's
// next block barrier publishes them.
__device__ __forceinline__ void store_points(const PointLoad &L, int count, float4 *c, float4 *s,
                                             float4 *v) {
    const int tid = threadIdx.x;
    if (tid < ((count + 3) & ~3)) {
        const bool real = tid < count;
        reinterpret_cast<float *>(c)[tid] = real ? L.c : 0.0f;
        reinterpret_cast<float *>(s)[tid] = real ? L.s : 0.0f;
        reinterpret_cast<float *>(v)[tid] = real ? L.v : __builtin_inff();
    }
}

// Inliers of hypothesis (hx, hy) among the first `tail` points of the tile (LDS
// broadcasts).
template <int N>
__device__ __forceinline__ uint32_t tail_count(const LaneTile<N> &sh, int tail, float hx, float hy,
                                               float tau) {
    uint32_t cnt = 0;
#pragma unroll 1
    for (int q = 0; q < (tail + 3) / 4; ++q) {
        const float4 c = sh.c[q], sn = sh.s[q], v = sh.v[q];
        const float cc[4] = {c.x, c.y, c.z, c.w}, ss[4] = {sn.x, sn.y, sn.z, sn.w};
        const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float e = __builtin_fmaf(-hy, ss[u], __builtin_fmaf(-hx, cc[u], vv[u]));
            cnt += __builtin_fabsf(e) < tau ? 1u : 0u;
        }
    }
    return cnt;
}

// A cluster's hypotheses: Philox key and the cluster index of the counter
// (the cluster's index within its own frame), and the index of its outputs.
struct ClusterId {
    int64_t out;       // index into the per-cluster outputs
    uint32_t local;    // counter word 1 of its hypotheses
    uint32_t key0, key1;
};

// Key of the wave's best hypothesis, the same in every lane: val = its count + 1
// (0: none), the lowest h among the largest; 0 when no lane has one.
__device__ __forceinline__ unsigned long long wave_best(uint32_t val, uint32_t h) {
    const uint32_t most = wave_max_u32(val);
    if (most == 0) return 0;
    const uint32_t low = ~wave_max_u32(val == most ? ~h : 0u);
    return ((unsigned long long)(most - 1u) << 32) | (0xFFFFFFFFull - low);
}

// The largest of the block's per-wave keys (LDS), the same in every thread.
template <int B>
__device__ __forceinline__ unsigned long long block_key(const unsigned long long *keys) {
    unsigned long long key = keys[0];
#pragma unroll
    for (int w = 1; w < B / kWave; ++w) key = keys[w] > key ? keys[w] : key;
    return uniform_u64(key);
}

// A cluster's key while other workgroups may merge into it (some value it had lately),
// the same in every lane.
__device__ __forceinline__ unsigned long long load_key(const unsigned long long *key) {
    return uniform_u64(__hip_atomic_load(key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// A cluster's key with every merge that came before, the same in every lane.
__device__ __forceinline__ unsigned long long read_key(unsigned long long *key) {
    unsigned long long k = 0;
    if (threadIdx.x % kWave == 0) k = atomicMax(key, 0ull);
    return uniform_u64(k);
}

// Merges a block's best key into the cluster's: a 64-bit atomic maximum, whose
// result does not depend on the order of the blocks.  Called by the whole block
// (the guard is wave-uniform: it may sit in a loop with barriers, see
// batch_score_kernel).
__device__ __forceinline__ void merge_key(unsigned long long *best_key, unsigned long long key,
                                          int wave, int lane) {
    if (wave == 0) {
        if (lane == 0 && key != 0) atomicMax(best_key, key);
    }
}

constexpr int kPruneHyp = 1024;  // hypotheses per workgroup, at most

// Workgroup LDS of the rows form.
template <int B>
struct RowsShared {
    float4 hyp[kPruneHyp / 2];  // (vx, vy) pairs, two per float4
    unsigned long long key[B / kWave];
    LaneTile<kLaneTile> tile;
};

// One scoring block: hypotheses [b B, b B + B) of one cluster, B threads.  Each
// thread draws and solves one hypothesis into LDS (drawn: they are there, at entry q B
// of its list); each wave then scores 64 of them against every point of the cluster: lanes = points over the cluster's full
// rows, lanes = hypotheses over its tail, or over the whole cluster when it has at
// most lanes_max (<= kLaneTile) points.  Returns the block's best (count, lowest
// index) key over its valid hypotheses, the same in every thread.  Called by all
// threads of the block, also from the persistent loop (every branch around a
// barrier is on a wave-uniform value).
template <int B, int kRows>
__device__ __forceinline__ unsigned long long score_block(Span sp, ClusterId id, int b, int q,
                                                          bool drawn, int32_t n_hyp,
                                                          const Points &pts, float tau, int rows_max,
                                                          int lanes_max, RowsShared<B> &sh,
                                                          int32_t *__restrict__ hyp_counts) {
    static_assert(kLaneTile <= B, "a thread stages a point");
    const int tid = threadIdx.x;
    const int64_t h = (int64_t)b * B + tid;
    if (!sp.ok || sp.n < 2) {
        if (hyp_counts != nullptr && h < n_hyp) hyp_counts[id.out * n_hyp + h] = 0;
        return 0;
    }
    const int tail = sp.n <= lanes_max ? (int)sp.n : lanes_tail(sp.n);  // the same for the block
    const float4 *hyp = sh.hyp + q * (B / 2);
    float2 own = make_float2(__builtin_nanf(""), __builtin_nanf(""));
    {
        // The tail points' loads go out before the hypothesis's seed loads and
        // are stored after its solve, so the two latencies overlap.
        PointLoad tl;
        if (tail > 0) tl = load_point(pts, sp.lo + sp.n - tail, tail);
        if (!drawn) {
            if (h < n_hyp) {
                const Hypothesis y = make_hypothesis(pts, sp, (uint32_t)h, id.local, id.key0, id.key1);
                own = make_float2((float)y.vx, (float)y.vy);  // NaN exactly when degenerate
            }
            reinterpret_cast<float2 *>(sh.hyp)[q * B + tid] = own;
        }
        if (tail > 0) store_points(tl, tail, sh.tile.c, sh.tile.s, sh.tile.v);
    }
    __syncthreads();

    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const int64_t h0 = (int64_t)b * B + wave * kWave;
    uint32_t val = 0;  // count + 1 of a valid hypothesis
    if (h0 < n_hyp) {
        const int nh = (int64_t)n_hyp - h0 < kWave ? (int)((int64_t)n_hyp - h0) : kWave;
        Span rows = sp;
        rows.n -= tail;
        uint32_t cnt = 0;
        if (rows.n > 0)
            cnt = score_cluster<kRows, true>(pts, rows, lane, hyp + wave * (kWave / 2), nh, tau,
                                             rows_max);
        // The lane's own hypothesis is re-read from LDS rather than kept in
        // registers through the scoring loop.
        own = reinterpret_cast<const float2 *>(hyp)[tid];
        cnt += tail_count(sh.tile, tail, own.x, own.y, tau);
        if (lane < nh) {
            if (hyp_counts != nullptr) hyp_counts[id.out * n_hyp + h] = (int32_t)cnt;
            if (!__builtin_isnan(own.x)) val = cnt + 1u;
        }
    }
    const unsigned long long key = wave_best(val, (uint32_t)h);
    if (lane == 0) sh.key[wave] = key;
    __syncthreads();
    return block_key<B>(sh.key);
}

// ---------------------------------------------------------------------------
// FP16 residual form of the scoring (batched form, clusters of at least
// Tuning::fp16_min points).  It selects exactly the hypothesis the float32
// form selects; only the work differs.
//
// Per workgroup (cluster, block of 256 hypotheses):
//   1. reference velocity r = (rx, ry): the block's hypothesis with the most
//      float32 inliers among the cluster's first kFp16Sample points;
//   2. every point of a pass holds half2 (cos, sin) (rounded toward zero) and
//      the float32 residual w = fma(-ry, sin, fma(-rx, cos, v_d)); hypothesis
//      h = (hx, hy) arrives as half2 -(hx - rx, hy - ry), and one
//      v_dot2_f32_f16 adds the two FP16 products to w in float32;
//   3. the FP16 count hi_h uses the widened threshold tau + B_h, where B_h
//      bounds |FP16 residual - float32 residual| at every point whose float32
//      residual is below tau, so hi_h >= the float32 count n_h;
//   4. the hypothesis with the largest (hi_h, lowest index) is counted exactly
//      in float32 (T = its n_h); every other hypothesis with hi_h >= T is
//      counted exactly too.  A hypothesis left out has n_h <= hi_h < T, so the
//      block's best exact key, merged with the same 64-bit atomic maximum, is
//      the float32 form's.
//
// Error bound (A = |hx - rx| + |hy - ry|, M = |hx| + |hy| + |rx| + |ry|, both
// in float32; u = 2^-24): for a point with |float32 residual| < tau, the
// terms are the rounding of w (about u (2|R| + 2A + M)), of -(h - r) to FP16
// (2^-11 A) and of (cos, sin) toward zero (2^-10 A, plus 2^-24 A for FP16
// subnormals), and the sums inside the dot product (at most 8u (2A + |R|));
// together below 2^-9 A + 2^-20 (tau + M + 1).  B_h takes twice that,
// 2^-8 A + 2^-18 (tau + M + 1), which also covers the float32 rounding of
// tau + B_h.  A hypothesis with A >= 2^14 (or not finite) is not converted:
// its FP16 row counts every finite point (threshold +inf), a valid upper bound.
// (cos, sin) below 2^-14 in magnitude may lose their value in the dot product
// if it flushes FP16 subnormals; that error, at most 2^-14 A, is inside 2^-8 A.
// ---------------------------------------------------------------------------

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int kFp16Sample = 4 * kWave;  // points of the reference-velocity sample
constexpr float kFp16MaxOffset = 16384.0f;

// (bits of half2 -(h - r), widened threshold) of one hypothesis; an invalid
// one (NaN) gets threshold 0, which no residual passes.
__device__ __forceinline__ float2 fp16_hypothesis(float hx, float hy, float rx, float ry,
                                                  float tau) {
    if (__builtin_isnan(hx) || __builtin_isnan(hy)) return make_float2(0.0f, 0.0f);
    float dx = hx - rx, dy = hy - ry;
    const float a = __builtin_fabsf(dx) + __builtin_fabsf(dy);
    if (!(a < kFp16MaxOffset)) return make_float2(0.0f, __builtin_inff());
    const float m = __builtin_fabsf(hx) + __builtin_fabsf(hy) + __builtin_fabsf(rx) +
                    __builtin_fabsf(ry);
    // An offset component below the smallest normal FP16 value is sent as 0 and
    // its magnitude (at most 2^-14 per point, |cos|, |sin| <= 1) joins the band,
    // so the bound holds whether or not the dot product keeps FP16 subnormals.
    float tiny = 0.0f;
    if (__builtin_fabsf(dx) < 0x1p-14f) {
        tiny += __builtin_fabsf(dx);
        dx = 0.0f;
    }
    if (__builtin_fabsf(dy) < 0x1p-14f) {
        tiny += __builtin_fabsf(dy);
        dy = 0.0f;
    }
    const float band = a * 0x1p-8f + (tau + m + 1.0f) * 0x1p-18f + 2.0f * tiny;
    const half2_t nd = half2_t{(_Float16)(-dx), (_Float16)(-dy)};
    return make_float2(__builtin_bit_cast(float, nd), tau + band);
}

// One hypothesis (nd = half2 -(h - r), threshold t) against four rows of
// points in the FP16 form: e = v_dot2_f32_f16(cs, nd) + w, each product in
// FP16 and the sum in float32, then |e| < t as four 64-lane masks; returns the
// number of set bits.  The VOP3P v_dot2_f32_f16 writes its own destination:
// the compiler's choice, the accumulating v_dot2c_f32_f16, overwrites w and so
// needs a copy of w for every row and hypothesis (three vector instructions
// per row instead of two).  One asm block, so that each compare issues three
// instructions after the dot product whose result it reads: gfx950 needs three
// wait states between a DOT instruction's write and another VALU instruction's
// read of that register.  Every lane must be active (the masks are ballots).
__device__ __forceinline__ uint32_t fp16_count4(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                float w0, float w1, float w2, float w3,
                                                uint32_t nd, float t) {
    float e0, e1, e2, e3;
    uint64_t m0, m1, m2, m3;
    asm("v_dot2_f32_f16 %0, %8, %12, %14\n\t"
        "v_dot2_f32_f16 %1, %9, %12, %15\n\t"
        "v_dot2_f32_f16 %2, %10, %12, %16\n\t"
        "v_dot2_f32_f16 %3, %11, %12, %17\n\t"
        "v_cmp_lt_f32_e64 %4, |%0|, %13\n\t"
        "v_cmp_lt_f32_e64 %5, |%1|, %13\n\t"
        "v_cmp_lt_f32_e64 %6, |%2|, %13\n\t"
        "v_cmp_lt_f32_e64 %7, |%3|, %13"
        : "=&v"(e0), "=&v"(e1), "=&v"(e2), "=&v"(e3), "=s"(m0), "=s"(m1), "=s"(m2), "=s"(m3)
        : "v"(c0), "v"(c1), "v"(c2), "v"(c3), "v"(nd), "v"(t), "v"(w0), "v"(w1), "v"(w2),
          "v"(w3));
    return (uint32_t)(__builtin_popcountll(m0) + __builtin_popcountll(m1) +
                      __builtin_popcountll(m2) + __builtin_popcountll(m3));
}

// score_rows in the FP16 form: returns hi of hypothesis q of the wave in lane q.
// R is a multiple of four; rows past the points are padding (w = +inf).
template <int R>
__device__ __forceinline__ uint32_t score_rows_fp16(const StagedPoint *__restrict__ chunk, int npts,
                                                    int lane, const float4 *hp, int ng, float rx,
                                                    float ry) {
    static_assert(R % 4 == 0, "rows come in blocks of four");
    uint32_t cs[R];
    float w[R];
    const uint32_t at = (uint32_t)lane * (uint32_t)sizeof(StagedPoint);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int len = npts - r * kWave;
        cs[r] = 0u;
        w[r] = __builtin_inff();
        if (lane < len) {
            const StagedPoint &q = row_point(chunk + r * kWave, at);
            cs[r] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(q.c, q.s));
            w[r] = __builtin_fmaf(-ry, q.s, __builtin_fmaf(-rx, q.c, q.v));
        }
    }
    uint32_t counts = 0;
    for (int g = 0; g < ng; ++g) {
        const float4 h0 = hp[2 * g], h1 = hp[2 * g + 1];
        const float hd[kHypGroup] = {h0.x, h0.z, h1.x, h1.z};
        const float ht[kHypGroup] = {h0.y, h0.w, h1.y, h1.w};
#pragma unroll
        for (int u = 0; u < kHypGroup; ++u) {
            const uint32_t nd = __builtin_bit_cast(uint32_t, hd[u]);
            uint32_t n = 0;
#pragma unroll
            for (int r = 0; r < R; r += 4)
                n += fp16_count4(cs[r], cs[r + 1], cs[r + 2], cs[r + 3], w[r], w[r + 1], w[r + 2],
                                 w[r + 3], nd, ht[u]);
            counts = (uint32_t)amdgcn_writelane((int)n, g * kHypGroup + u, (int)counts);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return counts;
}

// score_cluster in the FP16 form (a pass's rows rounded up to a multiple of
// four).
__device__ __forceinline__ uint32_t score_cluster_fp16(const Points &pts, Span sp, int lane,
                                                       const float4 *hp, int nh, int rows_max,
                                                       float rx, float ry) {
    const int ng = (nh + kHypGroup - 1) / kHypGroup;
    const int64_t end = sp.lo + sp.n;
    const int64_t pass = (int64_t)rows_max * kWave;
    uint32_t total = 0;
    for (int64_t base = sp.lo; base < end; base += pass) {
        const int64_t left = end - base;
        const int npts = (int)(left < pass ? left : pass);
        const int blocks = (npts + 4 * kWave - 1) / (4 * kWave);
        const StagedPoint *chunk = pts.staged + base;
        switch (blocks) {
#define RV_ROWS16(B)                                                                       \
    case B:                                                                                \
        total += score_rows_fp16<4 * B>(chunk, npts, lane, hp, ng, rx, ry);                 \
        break;
            RV_ROWS16(1) RV_ROWS16(2) RV_ROWS16(3) RV_ROWS16(4)
#undef RV_ROWS16
            default: break;
        }
    }
    return total;
}

// Workgroup LDS of the FP16 form.
struct Fp16Shared {
    float4 h32[kScoreBlock / 2];               // float32 (vx, vy) of the block's hypotheses
    float4 h16[kScoreBlock / 2];               // fp16_hypothesis() of each
    float4 list[kWave / 2];                    // hypotheses counted exactly, float32
    uint32_t part[kScoreBlock / kWave][kWave]; // per-wave partial exact counts
    uint32_t idx[kScoreBlock];                 // candidates: positions in the block
    unsigned long long key[kScoreBlock / kWave];
    uint32_t n_cand[kScoreBlock / kWave];
};

constexpr int kExactRows = 8;  // register rows per pass of the exact counts

__device__ __forceinline__ unsigned long long hyp_key(uint32_t count, int64_t h) {
    return ((unsigned long long)count << 32) | (0xFFFFFFFFull - (uint32_t)h);
}

// Small clusters score with lanes = hypotheses: with lanes = points a cluster of
// n < 64 points leaves 64 - n lanes of every compare idle and pays the
// per-hypothesis overhead on a single row.  The residual and the test are the
// rows form's, fma(-hy, s, fma(-hx, c, v_d)) and |.| < tau, so every count, and
// the block's key, is the same bit for bit.
constexpr int kDefaultLanesMax = 64;  // default Tuning::lanes_max
constexpr int kSingleLanesMax = 64;   // single-frame calls

// Exact float32 counts of the nl (<= 64) hypotheses in `list` (LDS) over the
// whole cluster; the block's waves share the cluster's rows.
// Lane q of every wave returns the count of list entry q.  Contains barriers.
template <int B>
__device__ __forceinline__ uint32_t exact_counts(Span sp, const Points &pts, float tau, int nl,
                                                 const float4 *list, uint32_t (*part_sums)[kWave],
                                                 int wave, int lane) {
    const int64_t rows = (sp.n + kWave - 1) / kWave;
    const int64_t r0 = rows * wave / (B / kWave);
    const int64_t r1 = rows * (wave + 1) / (B / kWave);
    const int64_t p1 = r1 * kWave < sp.n ? r1 * kWave : sp.n;
    Span part;
    part.lo = sp.lo + r0 * kWave;
    part.n = p1 - r0 * kWave;
    part.ok = true;
    part_sums[wave][lane] = score_cluster<kExactRows>(pts, part, lane, list, nl, tau, kExactRows);
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int w = 0; w < B / kWave; ++w) total += part_sums[w][lane];
    __syncthreads();
    return total;
}

// exact_counts in the FP16 form: upper bounds of the counts of the nl hypotheses
// in `list` (fp16_hypothesis pairs against (rx, ry)).
template <int B>
__device__ __forceinline__ uint32_t fp16_counts(Span sp, const Points &pts, int nl,
                                                const float4 *list, uint32_t (*part_sums)[kWave],
                                                int wave, int lane, float rx, float ry) {
    const int64_t rows = (sp.n + kWave - 1) / kWave;
    const int64_t r0 = rows * wave / (B / kWave);
    const int64_t r1 = rows * (wave + 1) / (B / kWave);
    const int64_t p1 = r1 * kWave < sp.n ? r1 * kWave : sp.n;
    Span part;
    part.lo = sp.lo + r0 * kWave;
    part.n = p1 - r0 * kWave;
    part.ok = true;
    part_sums[wave][lane] = score_cluster_fp16(pts, part, lane, list, nl, kExactRows, rx, ry);
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int w = 0; w < B / kWave; ++w) total += part_sums[w][lane];
    __syncthreads();
    return total;
}

// ---------------------------------------------------------------------------
// Large clusters: counting only the hypotheses that can still win.
//
// Only the hypothesis with the most inliers is kept, so a hypothesis need not
// be counted once its count is known to be below another's.  Per workgroup
// (one cluster, up to kPruneHyp hypotheses):
//   1. reference r: among the first 64 hypotheses the one with the most inliers in
//      a strided sample of the points;
//   2. one sweep over the cluster counts r exactly (T) and sorts the points
//      into a table of direction (kAngleBins<B>) x signed residual under r;
//   3. every hypothesis h gets an upper bound of its count from the table: a
//      point with direction u is an inlier of h only if its residual under r
//      lies within tau of (h - r).u, and over one direction bin (h - r).u
//      stays in a known interval, so h's inliers in the bin are at most the
//      bin's points in that interval widened by tau: two prefix-sum lookups;
//   4. the hypotheses with the largest bounds (one per wave) are counted, which
//      raises the best known count;
//   5. every hypothesis whose bound still reaches the best known (count, lowest
//      index) is counted in float32 over all points.
// A hypothesis left out has count <= bound and loses to a counted one, so the
// best key, and every output, is the full count's bit for bit.  (Calls that ask
// for every hypothesis's count take the full count.)
//
// With 20 to 40 % outliers about one hypothesis in eight reaches r's count in
// step 3 and one in twenty the best key in step 5.  What remains is per
// hypothesis: the draw and solve (about 230 vector instructions per 64
// hypotheses) and the bound (16 table lookups and about 170), against 3.7 per
// 64 hypotheses and point of the full count.  Scoring stage before and after on
// frames of equal clusters, 4.2M hypotheses: 4096 clusters of 512 points 152 and
// 78 us, 1024 of 2048 points 151 and 52 us; the 4096-cluster frame of 8 to 4096
// points 193 and 84 us; 64 clusters of 65,536 points at 4096 hypotheses 1.40 and
// 0.10 ms (0.27 ms in small workgroups, see long_clusters).
//
// Rounding.  A point with |float32 residual under h| < tau has an exact
// residual (of the float32 cos, sin, v_d and velocities) within
// 2^-24 (2 tau + |hy|) of it; its float32 residual under r is within
// 2^-24 (2 (tau + |hx - rx| + |hy - ry|) + |ry|) of the exact one; the float32
// evaluation of (h - r).u at a bin's centre, the bin's centre direction and the
// staged direction's length add at most 2^-21 (|hx - rx| + |hy - ry|).  All of
// it is below 2^-19 (tau + M), M = |hx| + |hy| + |rx| + |ry|; the interval is
// widened by 2^-18 (tau + M).
// ---------------------------------------------------------------------------

constexpr int kSample = 32;         // points of the sample

// Clusters of at least this many points in a long frame of few workgroups are deferred
// when the table would exclude too little (plan_score); the mark in such a cluster's key.
constexpr int64_t kDeferPoints = 1024;
constexpr uint32_t kGiveUpPoints = 2048;
constexpr unsigned long long kDeferred = 1ull << 63;

// When the table would exclude too little, every hypothesis is counted after all: when
// the reference holds fewer than `sample` of the 32 sampled points, seen before the
// table is made, or fewer than share / 64 of the cluster's points, seen after it.  The
// hypotheses are drawn already; what is lost are one or two sweeps.  Scoring stage in us
// at 1024 hypotheses: always with the table, by this rule, and before there was a table:
//   outliers             60 %            70 %             90 %
//   3177 of 330 points   85,  86,  92    140, 121, 92     190, 112, 93
//   2048 of 512 points   73,  75,  81    116,  99, 81     140, 100, 81
//   5242 of 200 points  100,  99, 109    158, 112, 110    225,  95, 109
// Small clusters (score_small is their other form) gain least from the table.  From 1024
// points on it still halves the time at 60 % (256 of 4096 points 63, 63, 97 us) and
// makes no difference at 70 % (98, 98, 97), and a workgroup that gives up by the chance of
// its sample alone sets the end of the call (4096 clusters of 8 to 4096 points at 60 %: 124
// us, 146 with the line of 1024 points for all): only the hopeless are told.  A few
// hypotheses are not given up either: the list's count shares the points between all
// waves (16 clusters of 4096 points, 64 hypotheses, 85 %: call 47 and 87 us).
// A long cluster that a single compute unit would be counting is given up sooner, since
// it is spread over the chip then (64 of 30,000 points 59, 56, 467 us; 374, 214, 468;
// 721, 214, 468 with the refit).
struct GiveUp {
    uint32_t sample, share;
};

// (enough: more than half of the workgroup's waves would have hypotheses to count.)
__device__ __forceinline__ GiveUp give_up(uint32_t n, bool enough, bool defer) {
    if (!enough) return {0, 0};
    if (n <= kLaneTile) return {13, 17};
    if (n < kDeferPoints) return {8, 17};
    if (defer) return {6, 20};
    if (n < kGiveUpPoints) return {6, 12};
    return {3, 0};
}

// Smallest cluster scored this way, by blocks of 256 hypotheses per workgroup
// (at least 1).  The table is made once per workgroup, so the more blocks share it
// the sooner the bound pays: with four from 128 points on (16,384 clusters of 128
// points at 1024 hypotheses: scoring stage 247 us counted in full, 212 us this
// way), with two a little later (32,768 clusters of 128 points at 512 hypotheses:
// 256 and 264 us), with one from about 320 points on (a frame of 1021 clusters in
// 3-degree windows: 37, 35 and 34 us with the line at 128, 192 and 320).
__host__ __device__ constexpr int prune_min(int rounds) {
    return rounds == 1 ? 320 : rounds == 2 ? 160 : 128;
}

// Direction bins.  A long cluster's time is its sweeps and counts, and its large
// workgroup (long_clusters) has the LDS for four times as many: 64 clusters of 65,536
// points, 1024 of their 4096 hypotheses per workgroup, 39 to count for 58 (modelled),
// call 180 us with 32 directions, 199 us with 16, 226 us with 8.  Twice the residual
// bins as well: 177 us, but 130 for 122 us at 128 clusters of 16,384 points.
template <int B>
constexpr int kAngleBins = B == kLongBlock ? 32 : 8;
constexpr int kResidualBins = 256;  // 128 per sign, 16 per octave of |e| + unit (residual_bin)
constexpr int kResidualRow = kResidualBins + 1;
constexpr float kPruneMaxSpeed = 1e15f;  // references beyond it are not used

template <int B>
struct PruneShared {
    float4 hyp[kPruneHyp / 2];  // (vx, vy) pairs
    LaneTile<kSample> sample;
    float4 dir[kAngleBins<B>];     // centre (cos, sin), half width w, w^2 / 2
    union {
        uint32_t hist[kAngleBins<B> * kResidualRow];
        struct {
            uint32_t part[B / kWave][kWave];
            float list[2 * kWave] __attribute__((aligned(16)));
            uint16_t idx[kPruneHyp];
            float half_list[2 * kWave] __attribute__((aligned(16)));  // FP16 form
            uint16_t kept[kWave];
        } count;
    } u;
    unsigned long long key[B / kWave];
    unsigned long long top_key[B / kWave];
    unsigned long long floor_key;
    float lo[B / kWave], hi[B / kWave];
    uint32_t n[B / kWave];
    uint32_t top[B / kWave];
};
static_assert(1024 / kWave <= kWave, "a lane per wave's top");

// Position of a direction on the circle, monotone in its angle over (-pi, pi]:
// s / (|c| + |s|) in the right half plane, continued to +-2 at the left.
__device__ __forceinline__ float direction_key(float c, float s) {
    const float y = s * __builtin_amdgcn_rcpf(__builtin_fabsf(c) + __builtin_fabsf(s));
    return c >= 0.0f ? y : __builtin_copysignf(2.0f, s) - y;
}

// The unit vector of a direction key.
__device__ __forceinline__ float2 key_direction(float q) {
    const float a = __builtin_fabsf(q);
    const float c = 1.0f - a;
    const float s = __builtin_copysignf(a <= 1.0f ? a : 2.0f - a, q);
    const float inv = __builtin_amdgcn_rsqf(c * c + s * s);
    return make_float2(c * inv, s * inv);
}

// Residual bin of e' = e sigma, with sigma the power of two that takes tau into
// [4, 8) (residual_scale): the octaves of |e'| + 2 in sixteen bins each, eight
// octaves, beyond them the last bin.  Monotone in e' (the float addition, the
// minimum and the bit pattern of a positive float are), so a window [lo, hi] of
// residuals holds only points of bins residual_bin(lo) to residual_bin(hi).
__device__ __forceinline__ int residual_bin(float e) {
    const float t = fminf(__builtin_fabsf(e) + 2.0f, 511.0f);
    // exponent field 128 to 135: its low bits and four of the mantissa
    const uint32_t k = (__builtin_bit_cast(uint32_t, t) >> 19) & 127u;
    return (int)(k ^ (uint32_t)(__builtin_bit_cast(int32_t, e) >> 31)) + kResidualBins / 2;
}

__device__ __forceinline__ float residual_scale(float tau) {
    const uint32_t exponent = (__builtin_bit_cast(uint32_t, tau) >> 23) & 255u;  // tau is normal
    return __builtin_bit_cast(float, (127u + 127u + 2u - exponent) << 23);
}

__device__ __forceinline__ float uniform_f(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

// body(point, in) for the block's share of a cluster's points, every thread one
// point in B, kSweepLoads of them loaded before the first is used (in: the point is
// one of the n; past the end the last one is loaded again).
// A large workgroup has the registers for eight (64 clusters of 65,536 points: 172 us
// with four ahead, 168 us with eight).
template <int B, typename Body>
__device__ __forceinline__ void sweep_points(const StagedPoint *points, uint32_t n,
                                             const Body &body) {
    constexpr int kSweepLoads = B == kLongBlock ? 8 : 4;
    for (uint32_t base = 0; base < n; base += kSweepLoads * B) {
        PointLoad u[kSweepLoads];
#pragma unroll
        for (int i = 0; i < kSweepLoads; ++i)
            u[i] = load_at(points, base + i * B + threadIdx.x, n);
#pragma unroll
        for (int i = 0; i < kSweepLoads; ++i)
            if (base + i * B < n) body(u[i], base + i * B + threadIdx.x < n);  // uniform
    }
}

// Scoring of hypotheses [h_first, h_first + nh), nh <= kPruneHyp, of a cluster
// with at least kWave points.  Returns the best key among the hypotheses, or,
// where a key of best_key (the cluster's so far, shared by its workgroups;
// nullptr: none) beats them all, some key not above it.  Called by all threads
// of the block, also from the persistent loop: every branch around a barrier is
// on a wave-uniform value.
// full: the table excludes too little (give_up) and nothing was counted; the
// hypotheses lie in LDS (sh.hyp, NaN for a degenerate pair and past the last).
// kHalf: the remaining hypotheses are first counted in the FP16 residual form (see
// below; r as its reference velocity), 64 at a time, and only those whose upper
// count still reaches the best key are counted in float32.
template <int B, bool kHalf = false>
__device__ __forceinline__ unsigned long long score_pruned(
    Span sp, ClusterId id, int64_t h_first, int nh, const Points &pts, float tau,
    PruneShared<B> &sh, const unsigned long long *best_key, bool defer, bool &full) {
    constexpr int kPruneRounds = kPruneHyp / B;
    constexpr int kDirs = kAngleBins<B>;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const uint32_t n = (uint32_t)sp.n;
    const int rounds = (nh + B - 1) / B;
    const StagedPoint *points = pts.staged + sp.lo;
    float2 *hyp = reinterpret_cast<float2 *>(sh.hyp);

    // The sample, spread over the cluster.
    if (wave == 0) {
        const PointLoad L = load_at(points, (uint32_t)(((uint64_t)lane * n) / kSample), n);
        store_points(L, kSample, sh.sample.c, sh.sample.s, sh.sample.v);
    }
    // Range of the points' directions.
    float qlo = __builtin_inff(), qhi = -__builtin_inff();
    sweep_points<B>(points, n, [&](const PointLoad &u, bool) {
        const float q = direction_key(u.c, u.s);  // NaN for a non-finite point (0, 0)
        qlo = fminf(qlo, q);
        qhi = fmaxf(qhi, q);
    });
    for (int i = tid; i < kDirs * kResidualRow; i += B) sh.u.hist[i] = 0;
    // The hypotheses, two at a time so that their seed loads overlap (NaN for a
    // degenerate pair and past the last).
    float2 own = make_float2(0.0f, 0.0f);  // the thread's first
    const float2 none = make_float2(__builtin_nanf(""), __builtin_nanf(""));
    if (kPruneRounds == 1 || rounds == 1) {
        const Hypothesis y =
            make_hypothesis(pts, sp, (uint32_t)(h_first + tid), id.local, id.key0, id.key1);
        own = tid < nh ? make_float2((float)y.vx, (float)y.vy) : none;
        hyp[tid] = own;
    } else {
        for (int q = 0; q < rounds; q += 2) {
            const int h0 = q * B + tid, h1 = h0 + B;
            const Seeds d0 = draw_seeds(pts, sp, (uint32_t)(h_first + h0), id.local, id.key0, id.key1);
            const Seeds d1 = draw_seeds(pts, sp, (uint32_t)(h_first + h1), id.local, id.key0, id.key1);
            const Hypothesis y0 = solve_seeds(pts, d0);
            const float2 f0 = h0 < nh ? make_float2((float)y0.vx, (float)y0.vy) : none;
            hyp[h0] = f0;
            if (q == 0) own = f0;
            if (q + 1 < rounds) {
                const Hypothesis y1 = solve_seeds(pts, d1);
                hyp[h1] = h1 < nh ? make_float2((float)y1.vx, (float)y1.vy) : none;
            }
        }
    }
    qlo = wave_min_f(qlo);
    qhi = wave_max_f(qhi);
    if (lane == 0) {
        sh.lo[wave] = qlo;
        sh.hi[wave] = qhi;
    }
    __syncthreads();

    // 1. Reference (the other waves have none: 64 hypotheses over 32 points leave as
    // many hypotheses after step 4 as 256 over 64).
    if (wave > 0) {
        if (lane == 0) sh.key[wave] = 0;
    } else {
        const uint32_t cnt = tail_count(sh.sample, kSample, own.x, own.y, tau);
        const bool usable = __builtin_fabsf(own.x) + __builtin_fabsf(own.y) < kPruneMaxSpeed;  // not NaN
        const unsigned long long key = wave_best(usable ? cnt + 1u : 0u, (uint32_t)tid);
        if (lane == 0) sh.key[wave] = key;
    }
    float q0 = sh.lo[0], q1 = sh.hi[0];
#pragma unroll
    for (int w = 1; w < B / kWave; ++w) {
        q0 = fminf(q0, sh.lo[w]);
        q1 = fmaxf(q1, sh.hi[w]);
    }
    const float width = fmaxf(q1 - q0, 1e-6f) * (1.0f / kDirs);
    if (tid < kDirs) {
        // A direction bin's centre and half width (asin x <= 1.05 x up to half
        // a radian: bins are narrower than 60 degrees), widened for the
        // rounding of direction_key.
        const float2 a = key_direction(q0 + tid * width);
        const float2 b = key_direction(tid == kDirs - 1 ? q1 : q0 + (tid + 1) * width);
        const float dx = b.x - a.x, dy = b.y - a.y;
        const float w = 0.53f * __builtin_amdgcn_sqrtf(dx * dx + dy * dy) + 0x1p-15f;
        const float mx = a.x + b.x, my = a.y + b.y;
        const float inv = __builtin_amdgcn_rsqf(mx * mx + my * my);
        sh.dir[tid] = make_float4(mx * inv, my * inv, w, 0.5f * w * w);
    }
    __syncthreads();
    unsigned long long ref = 0;
#pragma unroll
    for (int w = 0; w < B / kWave; ++w) ref = sh.key[w] > ref ? sh.key[w] : ref;
    ref = uniform_u64(ref);

    const GiveUp rule = give_up(n, nh > B / 2, B == kLongBlock && defer);
    full = ref == 0 || (uint32_t)(ref >> 32) < rule.sample;
    if (full) {
        __syncthreads();  // the caller puts other data there
        return 0;
    }

    unsigned long long best = 0;  // best known (count, hypothesis) key, the same in every lane
    uint32_t ub[kPruneRounds];
    float rx = 0.0f, ry = 0.0f;
    {
        // 2. Table of the points under r.
        const uint32_t r_local = 0xFFFFFFFFu - (uint32_t)ref;
        rx = uniform_f(hyp[r_local].x);
        ry = uniform_f(hyp[r_local].y);
        const float sigma = uniform_f(residual_scale(tau));
        const float scale = 1.0f / width;
        uint32_t t = 0;
        sweep_points<B>(points, n, [&](const PointLoad &u, bool in) {
            const float e = __builtin_fmaf(-ry, u.s, __builtin_fmaf(-rx, u.c, u.v));
            t += in && __builtin_fabsf(e) < tau ? 1u : 0u;
            int b = (int)((direction_key(u.c, u.s) - q0) * scale);
            b = b < kDirs - 1 ? b : kDirs - 1;
            b = b > 0 ? b : 0;
            if (in && u.v < __builtin_inff())
                atomicAdd(&sh.u.hist[b * kResidualRow + residual_bin(e * sigma)], 1u);
        });
        t = (uint32_t)wave_sum_i((int)t);
        if (lane == 0) sh.n[wave] = t;
        __syncthreads();
        t = sh.n[0];
#pragma unroll
        for (int w = 1; w < B / kWave; ++w) t += sh.n[w];
        best = uniform_u64(hyp_key(t, h_first + r_local));
        full = (uint32_t)(best >> 32) < (uint32_t)(((uint64_t)n * rule.share) >> 6);
        if (full) {
            __syncthreads();
            return 0;
        }
        // Prefix sums along each row: 32 threads per row, eight bins each.
        constexpr int kRowThreads = 32;
        static_assert(kDirs * kRowThreads <= B && kDirs * kRowThreads % kWave == 0 &&
                      kResidualBins == kRowThreads * 8, "one pass of whole waves");
        if (wave < kDirs * kRowThreads / kWave) {
            uint32_t *row =
                sh.u.hist + (tid / kRowThreads) * kResidualRow + (tid % kRowThreads) * 8;
            uint32_t x[8], sum = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                x[i] = sum;
                sum += row[i];
            }
            uint32_t incl = sum;
#pragma unroll
            for (int d = 1; d < kRowThreads; d <<= 1) {
                const uint32_t y = __shfl_up(incl, d, kRowThreads);
                if (tid % kRowThreads >= d) incl += y;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) row[i] = incl - sum + x[i];
            if (tid % kRowThreads == kRowThreads - 1) row[8] = incl;
        }
        __syncthreads();
        // 3. Bounds.
        float w2 = sh.dir[0].w;
#pragma unroll
        for (int b = 1; b < kDirs; ++b) w2 = fmaxf(w2, sh.dir[b].w);
#pragma unroll
        for (int q = 0; q < kPruneRounds; ++q) {
            ub[q] = 0;
            if (q < rounds) {
                const float2 h = hyp[q * B + tid];
                const float m = __builtin_fabsf(h.x) + __builtin_fabsf(h.y) + __builtin_fabsf(rx) +
                                __builtin_fabsf(ry);
                const float dx = (h.x - rx) * sigma, dy = (h.y - ry) * sigma;
                const float band = __builtin_fmaf(__builtin_fabsf(dx) + __builtin_fabsf(dy), w2,
                                                  (tau + 0x1p-18f * (tau + m)) * sigma);
                uint32_t bound = 0;
#pragma unroll 4
                for (int b = 0; b < kDirs; ++b) {
                    const float4 d = sh.dir[b];
                    const float f = __builtin_fmaf(dx, d.x, dy * d.y);
                    const float g = __builtin_fmaf(dy, d.x, -dx * d.y);
                    const float rad = __builtin_fmaf(__builtin_fabsf(g), d.z, band);
                    const uint32_t *row = sh.u.hist + b * kResidualRow;
                    bound += row[residual_bin(f + rad) + 1] - row[residual_bin(f - rad)];
                }
                // Beyond this magnitude the interval arithmetic may overflow.
                if (!(m < 2.0f * kPruneMaxSpeed)) bound = n;
                // r itself is already counted.
                ub[q] = __builtin_isnan(h.x) || (q == 0 && tid == (int)r_local) ? 0u : bound;
            }
        }
    }

    // 4. The largest bound of each wave's hypotheses above the best key known
    // (this workgroup's r, or another workgroup's of the same cluster).
    unsigned long long floor_key = best;
    if (best_key != nullptr) {
        const unsigned long long other = load_key(best_key);
        floor_key = other > best ? other : best;
    }
    unsigned long long top = 0;
    {
        uint32_t most = 0, at = 0;
#pragma unroll
        for (int q = 0; q < kPruneRounds; ++q) {
            if (ub[q] > most) {
                most = ub[q];
                at = (uint32_t)(q * B + tid);
            }
        }
        top = wave_best(most != 0 ? most + 1u : 0u, (uint32_t)h_first + at);
        top = top > floor_key ? top : 0ull;
    }
    // Into an array of its own: without a reference no barrier lies between the reads
    // of sh.key above and here.  From here on every wave goes by the first one's floor:
    // each loaded the cluster's key at its own moment, and what they keep together has
    // to be decided by one.
    if (lane == 0) sh.top_key[wave] = top;
    if (wave == 0) sh.floor_key = floor_key;  // the same value from every lane
    __syncthreads();  // also the last use of the table
    floor_key = uniform_u64(sh.floor_key);
    int nl = 0;
    {
        int before = 0;
#pragma unroll
        for (int w = 0; w < B / kWave; ++w) {
            const int has = sh.top_key[w] != 0 ? 1 : 0;
            before += w < wave ? has : 0;
            nl += has;
        }
        nl = __builtin_amdgcn_readfirstlane(nl);
        if (lane == 0 && top != 0) {
            const uint32_t h = 0xFFFFFFFFu - (uint32_t)top - (uint32_t)h_first;
            reinterpret_cast<float2 *>(sh.u.count.list)[before] = hyp[h];
            sh.top[before] = h;
        }
    }
    // 5. Exact counts: the tops, then every hypothesis whose bound still
    // reaches the best key, 64 per pass.
    uint32_t n_cand = 0, c0 = 0;
    bool tops = true;
    while (nl > 0) {
        __syncthreads();
        uint32_t h = 0;
        if (lane < nl) h = tops ? sh.top[lane] : sh.u.count.idx[c0 - kWave + lane];
        if constexpr (kHalf) {
            if (!tops) {
                const float2 own = reinterpret_cast<const float2 *>(sh.u.count.list)[lane];
                const bool near = __builtin_fabsf(rx) + __builtin_fabsf(ry) < kFp16MaxOffset;
                const float fx = near ? rx : 0.0f, fy = near ? ry : 0.0f;
                reinterpret_cast<float2 *>(sh.u.count.half_list)[lane] =
                    fp16_hypothesis(own.x, own.y, fx, fy, tau);  // the same from every wave
                __syncthreads();
                const uint32_t hi = fp16_counts<B>(
                    sp, pts, nl, reinterpret_cast<const float4 *>(sh.u.count.half_list),
                    sh.u.count.part, wave, lane, fx, fy);
                const bool keep = lane < nl && hyp_key(hi, h_first + h) > floor_key;
                const uint64_t m = __builtin_amdgcn_ballot_w64(keep);  // the same in every wave
                if (wave == 0) {
                    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    if (keep) {
                        reinterpret_cast<float2 *>(sh.u.count.list)[rank] = own;
                        sh.u.count.kept[rank] = (uint16_t)h;
                    }
                }
                nl = __builtin_popcountll(m);
                __syncthreads();
                h = lane < nl ? sh.u.count.kept[lane] : 0u;
            }
        }
        const uint32_t cnt = exact_counts<B>(sp, pts, tau, nl,
                                             reinterpret_cast<const float4 *>(sh.u.count.list),
                                             sh.u.count.part, wave, lane);
        const unsigned long long k = wave_best(lane < nl ? cnt + 1u : 0u, (uint32_t)h_first + h);
        best = k > best ? k : best;
        floor_key = best > floor_key ? best : floor_key;
        if (tops) {
            tops = false;
            uint32_t mine = 0;
            uint64_t masks[kPruneRounds];
#pragma unroll
            for (int q = 0; q < kPruneRounds; ++q) {
                const unsigned long long kq =
                    ub[q] != 0 ? hyp_key(ub[q], h_first + q * B + tid) : 0ull;
                masks[q] = __builtin_amdgcn_ballot_w64(kq > floor_key && kq != top);
                mine += (uint32_t)__builtin_popcountll(masks[q]);
            }
            if (lane == 0) sh.n[wave] = mine;
            __syncthreads();
            uint32_t at = 0;
            n_cand = 0;
#pragma unroll
            for (int w = 0; w < B / kWave; ++w) {
                const uint32_t x = sh.n[w];
                at += w < wave ? x : 0u;
                n_cand += x;
            }
            n_cand = __builtin_amdgcn_readfirstlane(n_cand);
#pragma unroll
            for (int q = 0; q < kPruneRounds; ++q) {
                const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(masks[q] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)masks[q], 0u));
                if ((masks[q] >> lane) & 1) sh.u.count.idx[at + rank] = (uint16_t)(q * B + tid);
                at += (uint32_t)__builtin_popcountll(masks[q]);
            }
            __syncthreads();
        }
        const uint32_t rest = n_cand > c0 ? n_cand - c0 : 0u;
        nl = rest < (uint32_t)kWave ? (int)rest : kWave;
        if (tid < nl) reinterpret_cast<float2 *>(sh.u.count.list)[tid] = hyp[sh.u.count.idx[c0 + tid]];
        c0 += kWave;
    }
    return best;
}

// ---------------------------------------------------------------------------
// Small clusters, every hypothesis of the workgroup at once: lanes = hypotheses,
// each thread with up to four of them, the cluster's points broadcast from LDS.  A
// point's three broadcasts serve them all (with one hypothesis per thread the
// LDS, not the vector unit, set the rate: 15 cycles per point and 64 hypotheses).
// The compare, which issues at half the rate of an FMA, is a third FMA instead:
// (tau - |e|) 2^k with the result clamped to [0, 1] is exactly 1.0 when |e| < tau
// and 0 otherwise (NaN clamps to 0), for k such that one unit in the last place of
// tau times 2^k is at least 1; the product and tau 2^k are exact and the sum is
// rounded once, so its sign is that of tau - |e|.  The ones are added as integers,
// three operands an instruction, and their sum names the count: m times the bit
// pattern of 1.0f is 127 m 2^23, and 127 is odd.  The residual e is the rows form's,
// so every count is the same bit for bit.
// ---------------------------------------------------------------------------

constexpr uint32_t kInverse127 = 383;  // 127 * 383 = 1 mod 512: counts up to 511
static_assert((127u * kInverse127) % 512u == 1u && kLaneTile < 512, "counts are recovered mod 512");

template <int B>
struct SmallShared {
    float4 hyp[kPruneHyp / 2];
    LaneTile<kLaneTile> tile;
    unsigned long long key[B / kWave];
};

template <int H>
__device__ __forceinline__ void count_small(const LaneTile<kLaneTile> &tile, int n,
                                            const float2 *hyp, int stride, float tau,
                                            uint32_t (&count)[4]) {
    const uint32_t exponent = (__builtin_bit_cast(uint32_t, tau) >> 23) & 255u;  // tau is normal
    const float scale = __builtin_bit_cast(float, (127u + 127u + 25u - exponent) << 23);
    const float limit = tau * scale;
    float hx[H], hy[H];
    uint32_t sum[H];
#pragma unroll
    for (int k = 0; k < H; ++k) {
        hx[k] = hyp[k * stride].x;
        hy[k] = hyp[k * stride].y;
        sum[k] = 0;
    }
#pragma unroll 1
    for (int q = 0; q < (n + 3) / 4; ++q) {
        const float4 c = tile.c[q], sn = tile.s[q], v = tile.v[q];
        const float cc[4] = {c.x, c.y, c.z, c.w}, ss[4] = {sn.x, sn.y, sn.z, sn.w};
        const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < H; ++k) {
            uint32_t one[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float e = __builtin_fmaf(-hy[k], ss[u], __builtin_fmaf(-hx[k], cc[u], vv[u]));
                one[u] = __builtin_bit_cast(
                    uint32_t, __builtin_amdgcn_fmed3f(
                                  __builtin_fmaf(-__builtin_fabsf(e), scale, limit), 0.0f, 1.0f));
            }
            sum[k] = sum[k] + one[0] + one[1];
            sum[k] = sum[k] + one[2] + one[3];
        }
    }
#pragma unroll
    for (int k = 0; k < H; ++k) count[k] = ((sum[k] >> 23) * kInverse127) & 511u;
}

// Hypotheses [h_first, h_first + nh), nh <= kPruneHyp, of a cluster with 2 <= n <=
// kLaneTile points; tau in the range of prune_from.  The best key, the same in
// every thread.  Called by all threads of the block, also from the persistent loop.
template <int B>
__device__ __forceinline__ unsigned long long score_small(Span sp, ClusterId id, int64_t h_first,
                                                          int nh, bool drawn, int32_t n_hyp,
                                                          const Points &pts, float tau,
                                                          SmallShared<B> &sh,
                                                          int32_t *__restrict__ hyp_counts) {
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const int n = (int)sp.n, rounds = (nh + B - 1) / B;
    float2 *hyp = reinterpret_cast<float2 *>(sh.hyp);
    const PointLoad tl = load_point(pts, sp.lo, n);
#pragma unroll 1
    for (int q = drawn ? rounds : 0; q < rounds; ++q) {
        const int hl = q * B + tid;
        const Hypothesis y =
            make_hypothesis(pts, sp, (uint32_t)(h_first + hl), id.local, id.key0, id.key1);
        const float qnan = __builtin_nanf("");
        hyp[hl] = hl < nh ? make_float2((float)y.vx, (float)y.vy) : make_float2(qnan, qnan);
    }
    store_points(tl, n, sh.tile.c, sh.tile.s, sh.tile.v);
    __syncthreads();
    uint32_t val = 0, h = 0;  // the thread's best: count + 1 of a valid hypothesis, its index
#pragma unroll 1
    for (int q0 = 0; q0 < rounds; q0 += 4) {
        uint32_t count[4] = {0, 0, 0, 0};
        const int left = rounds - q0;
        if (left == 1)
            count_small<1>(sh.tile, n, hyp + q0 * B + tid, B, tau, count);
        else if (left == 2)
            count_small<2>(sh.tile, n, hyp + q0 * B + tid, B, tau, count);
        else
            count_small<4>(sh.tile, n, hyp + q0 * B + tid, B, tau, count);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int hl = (q0 + k) * B + tid;
            if (q0 + k < rounds && hl < nh) {
                if (hyp_counts != nullptr) hyp_counts[id.out * n_hyp + h_first + hl] = (int32_t)count[k];
                if (count[k] + 1u > val && !__builtin_isnan(hyp[hl].x)) {
                    val = count[k] + 1u;
                    h = (uint32_t)h_first + (uint32_t)hl;
                }
            }
        }
    }
    const unsigned long long key = wave_best(val, h);
    if (lane == 0) sh.key[wave] = key;
    __syncthreads();
    return block_key<B>(sh.key);
}

// Streams of a cluster's sums in the refit, per-lane sums of its waves (refit_cluster).
constexpr int kRefitStreams = 4;
constexpr int64_t kRefitLongPoints = 8192;

template <int kWaves>
struct RefitShared {
    double sum[kWaves][5][kWave];
    int cnt[kWaves][2][kWave];
};

// Workgroup LDS of the scoring forms and of the refit behind them: a workgroup uses one
// at a time.
template <int B>
struct ScoreShared {
    static constexpr size_t kBytes = sizeof(PruneShared<B>) > sizeof(RefitShared<B / kWave>)
                                         ? sizeof(PruneShared<B>) : sizeof(RefitShared<B / kWave>);
    static_assert(sizeof(RowsShared<B>) <= kBytes && sizeof(Fp16Shared) <= kBytes &&
                  sizeof(SmallShared<B>) <= kBytes, "the largest");
    alignas(16) unsigned char bytes[kBytes];
    __device__ RowsShared<B> &rows() { return *reinterpret_cast<RowsShared<B> *>(bytes); }
    __device__ Fp16Shared &fp16() { return *reinterpret_cast<Fp16Shared *>(bytes); }
    __device__ SmallShared<B> &small() { return *reinterpret_cast<SmallShared<B> *>(bytes); }
    __device__ PruneShared<B> &prune() { return *reinterpret_cast<PruneShared<B> *>(bytes); }
    __device__ RefitShared<B / kWave> &refit() { return *reinterpret_cast<RefitShared<B / kWave> *>(bytes); }
};

// Scoring of hypotheses [h_first, h_first + nh) of one cluster by one
// workgroup (h_first a multiple of B), in the form its size asks for; the best
// key, the same in every thread.  small_max: clusters of at most this many points
// (and at least two) take score_small; prune: clusters of at least this many points
// count only possible winners (half: behind the FP16 form); where that excludes too
// little, those up to the tile's size take score_small (unless small_max is 0), and
// with `defer` those of kDeferPoints points or more get kDeferred for a key; otherwise
// clusters of at most lanes_max points take lanes = hypotheses and the others
// lanes = points.
template <int B, int kRows, bool kFp16 = false>
__device__ __forceinline__ unsigned long long score_hypotheses(
    Span sp, ClusterId id, int64_t h_first, int nh, int32_t n_hyp, const Points &pts, float tau,
    int rows_max, int lanes_max, int small_max, int64_t prune, bool half, bool defer,
    ScoreShared<B> &sh,
    const unsigned long long *best_key, int32_t *__restrict__ hyp_counts) {
    bool drawn = false;  // the hypotheses lie in LDS
    if (sp.n >= prune && sp.n > small_max) {
        unsigned long long key;
        if (kFp16 && half)
            key = score_pruned<B, kFp16>(sp, id, h_first, nh, pts, tau, sh.prune(), best_key, defer, drawn);
        else
            key = score_pruned<B>(sp, id, h_first, nh, pts, tau, sh.prune(), best_key, defer, drawn);
        if (!drawn) return key;
        if (B == kLongBlock && defer && sp.n >= kDeferPoints) return kDeferred;
        if (small_max > 0 && sp.n <= kLaneTile) small_max = kLaneTile;
    }
    if (sp.n >= 2 && sp.n <= small_max)
        return score_small<B>(sp, id, h_first, nh, drawn, n_hyp, pts, tau, sh.small(), hyp_counts);
    const int b0 = (int)(h_first / B), blocks = (nh + B - 1) / B;
    unsigned long long best = 0;
    for (int q = 0; q < blocks; ++q) {
        const unsigned long long key = score_block<B, kRows>(sp, id, b0 + q, q, drawn, n_hyp, pts, tau,
                                                      rows_max, lanes_max, sh.rows(), hyp_counts);
        best = key > best ? key : best;
    }
    return best;
}

// One scoring block in the FP16 form (sp.ok and sp.n >= 2; called from the
// persistent loop: every branch around a barrier is on a wave-uniform value).
// hyp_counts, when requested, receives hi_h.
__device__ __forceinline__ void score_block_fp16(Span sp, ClusterId id, int b, int32_t n_hyp,
                                                 const Points &pts, float tau, int rows_max,
                                                 Fp16Shared &sh,
                                                 unsigned long long *__restrict__ best_key,
                                                 int32_t *__restrict__ hyp_counts) {
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)b * kScoreBlock;
    const int64_t h = base + tid;
    float hx = __builtin_nanf(""), hy = __builtin_nanf("");
    if (h < n_hyp) {
        const Hypothesis hyp = make_hypothesis(pts, sp, (uint32_t)h, id.local, id.key0, id.key1);
        hx = (float)hyp.vx;
        hy = (float)hyp.vy;
    }
    float2 *h32 = reinterpret_cast<float2 *>(sh.h32);
    h32[tid] = make_float2(hx, hy);
    __syncthreads();

    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const int64_t w0 = base + wave * kWave;
    const int nh = w0 < n_hyp ? ((int64_t)n_hyp - w0 < kWave ? (int)((int64_t)n_hyp - w0) : kWave)
                              : 0;

    // 1. Reference velocity from the sample.
    Span sample = sp;
    sample.n = sp.n < kFp16Sample ? sp.n : kFp16Sample;
    unsigned long long key = 0;
    if (nh > 0) {
        const uint32_t cnt = score_cluster<kFp16Sample / kWave>(
            pts, sample, lane, sh.h32 + wave * (kWave / 2), nh, tau, kFp16Sample / kWave);
        if (lane < nh && !__builtin_isnan(h32[tid].x)) key = hyp_key(cnt, base + tid);
    }
    key = wave_max_u64(key);
    if (lane == 0) sh.key[wave] = key;
    __syncthreads();
    unsigned long long ref = 0;
#pragma unroll
    for (int w = 0; w < kScoreBlock / kWave; ++w) ref = sh.key[w] > ref ? sh.key[w] : ref;
    ref = uniform_u64(ref);
    float rx = 0.0f, ry = 0.0f;
    if (ref != 0) {
        const float2 r = h32[(0xFFFFFFFFu - (uint32_t)ref) - (uint32_t)base];
        if (__builtin_fabsf(r.x) + __builtin_fabsf(r.y) < kFp16MaxOffset) {
            rx = r.x;
            ry = r.y;
        }
    }
    // The same value in every lane: kept in scalar registers.
    rx = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, rx)));
    ry = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, ry)));
    reinterpret_cast<float2 *>(sh.h16)[tid] = fp16_hypothesis(hx, hy, rx, ry, tau);
    __syncthreads();

    // 2-3. FP16 upper-bound counts (the lane's own hypothesis is re-read from
    // LDS afterwards rather than kept in registers through the loop).
    uint32_t hi = 0;
    if (nh > 0) hi = score_cluster_fp16(pts, sp, lane, sh.h16 + wave * (kWave / 2), nh, rows_max, rx, ry);
    const bool valid = lane < nh && !__builtin_isnan(h32[tid].x);
    // A hypothesis without a finite widened threshold (offset beyond the FP16
    // range) counted every finite point: its hi says nothing about its count.
    const bool wide = valid && !(reinterpret_cast<const float2 *>(sh.h16)[tid].y < __builtin_inff());
    if (hyp_counts != nullptr && lane < nh) hyp_counts[id.out * n_hyp + base + tid] = (int32_t)hi;
    key = valid && !wide ? hyp_key(hi, base + tid) : 0ull;
    key = wave_max_u64(key);
    const uint64_t wide_mask = __builtin_amdgcn_ballot_w64(wide);
    if (lane == 0) {
        sh.key[wave] = key;
        sh.n_cand[wave] = (uint32_t)__builtin_popcountll(wide_mask);
    }
    __syncthreads();
    unsigned long long top = 0;
    uint32_t wide_before = 0, n_wide = 0;
#pragma unroll
    for (int w = 0; w < kScoreBlock / kWave; ++w) {
        top = sh.key[w] > top ? sh.key[w] : top;
        const uint32_t c = sh.n_cand[w];
        wide_before += w < wave ? c : 0u;
        n_wide += c;
    }
    top = uniform_u64(top);
    n_wide = __builtin_amdgcn_readfirstlane(n_wide);
    if (top == 0 && n_wide == 0) return;  // no valid hypothesis in this block

    // 4. Exact float32 counts.  First pass: the hypothesis with the largest
    // (hi, lowest index) among those with a finite threshold (T = its exact
    // count) together with the hypotheses without one, up to 64 in all.  Then
    // every other valid hypothesis with hi >= T, 64 per pass.  A hypothesis
    // left out has n_h <= hi_h < T, so the best exact key is the float32 form's.
    const uint32_t has_top = top != 0 ? 1u : 0u;
    const uint32_t h_top = 0xFFFFFFFFu - (uint32_t)top;
    const uint32_t wide_rank =
        __builtin_amdgcn_mbcnt_hi((uint32_t)(wide_mask >> 32),
                                  __builtin_amdgcn_mbcnt_lo((uint32_t)wide_mask, 0u));
    const uint32_t slot = has_top + wide_before + wide_rank;
    const bool first = wide && slot < (uint32_t)kWave;  // counted in the first pass
    if (first) {
        reinterpret_cast<float2 *>(sh.list)[slot] = h32[tid];
        sh.idx[slot] = (uint32_t)tid;
    }
    if (tid == 0 && has_top) {
        reinterpret_cast<float2 *>(sh.list)[0] = h32[h_top - (uint32_t)base];
        sh.idx[0] = h_top - (uint32_t)base;
    }
    __syncthreads();
    const uint32_t n1 = has_top + n_wide < (uint32_t)kWave ? has_top + n_wide : (uint32_t)kWave;
    const uint32_t c1 = exact_counts<kScoreBlock>(sp, pts, tau, (int)n1, sh.list, sh.part, wave, lane);
    const uint32_t t_exact = has_top ? __builtin_amdgcn_readfirstlane(c1) : 0u;
    unsigned long long best = lane < (int)n1 ? hyp_key(c1, base + sh.idx[lane]) : 0ull;
    best = wave_max_u64(best);
    const bool cand = valid && !first && (!has_top || (uint32_t)(base + tid) != h_top) &&
                      hi >= t_exact;
    const uint64_t m = __builtin_amdgcn_ballot_w64(cand);
    if (lane == 0) sh.n_cand[wave] = (uint32_t)__builtin_popcountll(m);
    __syncthreads();
    uint32_t before = 0, n_cand = 0;
#pragma unroll
    for (int w = 0; w < kScoreBlock / kWave; ++w) {
        const uint32_t c = sh.n_cand[w];
        before += w < wave ? c : 0u;
        n_cand += c;
    }
    n_cand = __builtin_amdgcn_readfirstlane(n_cand);
    if (cand) {
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        sh.idx[before + rank] = (uint32_t)tid;
    }
    __syncthreads();
    for (uint32_t c0 = 0; c0 < n_cand; c0 += kWave) {
        const int nl = n_cand - c0 < (uint32_t)kWave ? (int)(n_cand - c0) : kWave;
        if (tid < nl) reinterpret_cast<float2 *>(sh.list)[tid] = h32[sh.idx[c0 + tid]];
        __syncthreads();
        const uint32_t cnt = exact_counts<kScoreBlock>(sp, pts, tau, nl, sh.list, sh.part, wave, lane);
        unsigned long long k2 = 0;
        if (lane < nl) k2 = hyp_key(cnt, base + sh.idx[c0 + lane]);
        k2 = wave_max_u64(k2);
        best = k2 > best ? k2 : best;
    }
    if (wave == 0) {
        if (lane == 0) atomicMax(&best_key[id.out], best);
    }
}

struct Outputs {
    float *vx, *vy, *heading;
    int32_t *n_inliers;
    uint8_t *status;
    int32_t *n_near, *best, *hyp_counts;
    uint32_t *bits;
};

__device__ __forceinline__ void write_failed(const Outputs &o, int64_t k, uint8_t st) {
    const float qnan = __builtin_nanf("");
    o.vx[k] = qnan;
    o.vy[k] = qnan;
    o.heading[k] = qnan;
    o.n_inliers[k] = 0;
    o.status[k] = st;
    if (o.n_near) o.n_near[k] = 0;
    if (o.best) o.best[k] = -1;
}

// A cluster's results from its inliers' normal-equation sums.
__device__ __forceinline__ void write_refit(const Outputs &o, int64_t k, uint32_t hbest, int n_in,
                                            int n_near, double scc, double scs, double sss,
                                            double scv, double ssv) {
    o.n_inliers[k] = n_in;
    if (o.n_near) o.n_near[k] = n_near;
    if (o.best) o.best[k] = (int32_t)hbest;
    const double det = scc * sss - scs * scs;
    if (n_in < 2 || !(det > 0.0)) {
        const float qnan = __builtin_nanf("");
        o.vx[k] = qnan;
        o.vy[k] = qnan;
        o.heading[k] = qnan;
        o.status[k] = RV_CLUSTER_SINGULAR_REFIT;
        return;
    }
    const double fvx = (sss * scv - scs * ssv) / det;
    const double fvy = (scc * ssv - scs * scv) / det;
    o.vx[k] = (float)fvx;
    o.vy[k] = (float)fvy;
    o.heading[k] = (float)atan2(fvy, fvx);
    o.status[k] = RV_CLUSTER_OK;
}

// FP64 sums of a refit, per lane.
struct RefitSums {
    double scc = 0.0, scs = 0.0, sss = 0.0, scv = 0.0, ssv = 0.0;
    int n_in = 0, n_near = 0;
};

// Re-classification of 64 points [p0, p0 + 64) of a cluster under h* (one wave,
// wave-uniform call): lane point p0 + lane counts when it is one of the cluster's and
// its v_d is finite (+inf marks a non-finite point); the block's ballot goes to the
// two or three words of the frame-wide mask that it lies in.  v and cs are loaded
// by the caller, so that the loads of several blocks are in flight together.
__device__ __forceinline__ void refit_points(int64_t p0, bool in_range, float v, double2 cs,
                                             const Hypothesis &hy, double dtau, RefitSums &a,
                                             const Outputs &o, int lane) {
    bool inlier = false;
    if (in_range && isfinite(v)) {
        const double c = cs.x, s = cs.y, dv = v;
        const double res = fabs(dv - hy.vx * c - hy.vy * s);
        a.n_near += fabs(res - dtau) <= RV_NEAR_TAU_WINDOW ? 1 : 0;
        if (res < dtau) {
            inlier = true;
            a.n_in += 1;
            a.scc += c * c;
            a.scs += c * s;
            a.sss += s * s;
            a.scv += c * dv;
            a.ssv += s * dv;
        }
    }
    if (o.bits != nullptr) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(inlier);
        if (lane == 0) {
            // A word holds no bit beyond the cluster's last point, so none outside the
            // mask is touched.
            const int sh = (int)(p0 & 31);
            const uint64_t low = m << sh;
            const uint32_t w0 = (uint32_t)low, w1 = (uint32_t)(low >> 32);
            const uint32_t w2 = sh != 0 ? (uint32_t)(m >> (64 - sh)) : 0u;
            if (w0) atomicOr(&o.bits[p0 >> 5], w0);
            if (w1) atomicOr(&o.bits[(p0 >> 5) + 1], w1);
            if (w2) atomicOr(&o.bits[(p0 >> 5) + 2], w2);
        }
    }
}

// One point of a wave's 64-point block from p0 on, loaded from a clamped, always
// valid index.
struct RefitLoad {
    StagedPoint p;
    StagedLow low;
    bool in;
};

__device__ __forceinline__ RefitLoad refit_load(Span sp, int64_t p0, const Points &pts, int lane) {
    const int64_t p = p0 + lane;
    RefitLoad L;
    L.in = p < sp.lo + sp.n;
    const int64_t at = L.in ? p : sp.lo;
    L.p = pts.staged[at];
    L.low = pts.low[at];
    return L;
}

// Sum over the wave in the fixed tree of lane distances 32, 16, ..., 1, all sums
// together, one distance per iteration of a rolled loop (code size: see
// refit_cluster).
__device__ __forceinline__ void wave_sum_all(RefitSums &a) {
#pragma unroll 1
    for (int o = kWave / 2; o > 0; o >>= 1) {
        a.scc += __shfl_xor(a.scc, o, kWave);
        a.scs += __shfl_xor(a.scs, o, kWave);
        a.sss += __shfl_xor(a.sss, o, kWave);
        a.scv += __shfl_xor(a.scv, o, kWave);
        a.ssv += __shfl_xor(a.ssv, o, kWave);
        a.n_in += __shfl_xor(a.n_in, o, kWave);
        a.n_near += __shfl_xor(a.n_near, o, kWave);
    }
}

__device__ __forceinline__ void add_sums(RefitSums &a, const RefitSums &b) {
    a.scc += b.scc;
    a.scs += b.scs;
    a.sss += b.sss;
    a.scv += b.scv;
    a.ssv += b.ssv;
    a.n_in += b.n_in;
    a.n_near += b.n_near;
}

// Refit of one cluster by `waves` waves (1, 4 or 16: all of a workgroup's; `wave` is
// this one's index among them): the kept hypothesis (from its best key), FP64
// re-classification of every point under it, least-squares refit on its inliers
// (Sec. 3.2, Eq. 7, Alg. 2: normal equations A^T A v = A^T v_d) and heading
// atan2(vy, vx) (Eq. 8).
//
// The order of the sums follows from the cluster's own points alone, whatever runs
// them, so a cluster has the same bits in a frame, a part of it, a batch of any size,
// and in every kernel that refits.  Per lane the 64-point blocks, counted from the
// cluster's first point, form kRefitStreams streams (every fourth block each), or from
// kRefitLongPoints points on sixteen; stream i + 4, i + 8 and i + 12 are added to stream i,
// then streams 0 to 3 in order, then the lanes in a fixed tree.  A wave walks its streams one
// after the other: one wave all four, one of four waves one or four, one of sixteen one.
//
// What bounds it on a few clusters is the code: every compute unit that runs it
// once fetches each of its lines once, at more than a hundred cycles a line.  So
// the sums and the point loop are rolled and the workgroup shapes share one copy.
// Wave-uniform branches only around the barriers.
template <int kWaves>
__device__ __forceinline__ void refit_cluster(Span sp, ClusterId id, unsigned long long best,
                                              const Points &pts, float tau, const Outputs &o,
                                              int wave, int waves, RefitShared<kWaves> &sh) {
    const int lane = threadIdx.x % kWave;
    const int64_t k = id.out;
    if (!sp.ok || sp.n < 2 || best == 0) {
        if (wave == 0) {
            if (lane == 0)
                write_failed(o, k, !sp.ok ? RV_CLUSTER_BAD_OFFSETS
                                          : sp.n < 2 ? RV_CLUSTER_TOO_FEW_POINTS
                                                     : RV_CLUSTER_ALL_DEGENERATE);
        }
        return;
    }
    const int streams = sp.n >= kRefitLongPoints ? 4 * kRefitStreams : kRefitStreams;
    const bool shared = waves > 1;
    // Where there are more waves than streams, the others only come to the barriers.
    constexpr bool kMore = kWaves > kRefitStreams;
    if (kMore && waves > streams) waves = streams;
    const uint32_t hbest = 0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull);
    RefitSums a;
    if (!kMore || wave < waves) {
        const int64_t end = sp.lo + sp.n, stride = (int64_t)streams * kWave;
        int stream = wave;  // of the block after p
        // The block after the one at p: the next of its stream, then the wave's next stream.
        const auto after = [&](int64_t p) {
            p += stride;
            if (p >= end && stream + waves < streams) {
                stream += waves;
                p = sp.lo + (int64_t)stream * kWave;
            }
            return p;
        };
        // Two blocks' loads in flight while the two before them are summed (the first
        // pair during the solve).
        int64_t p0 = sp.lo + (int64_t)wave * kWave, p1 = after(p0);
        RefitLoad a0 = refit_load(sp, p0, pts, lane), a1 = refit_load(sp, p1, pts, lane);
        const Hypothesis hy = make_hypothesis(pts, sp, hbest, id.local, id.key0, id.key1);
        RefitSums stream_sums;
#pragma unroll 1
        while (p0 < end) {
            const int64_t p2 = p1 < end ? after(p1) : p1;
            const RefitLoad b0 = refit_load(sp, p2, pts, lane);
            const int64_t p3 = p2 < end ? after(p2) : p2;
            const RefitLoad b1 = refit_load(sp, p3, pts, lane);
            refit_points(p0, a0.in, a0.p.v, cs64(a0.p, a0.low), hy, (double)tau, stream_sums, o, lane);
            if (p1 != p0 + stride) {
                add_sums(a, stream_sums);
                stream_sums = RefitSums();
            }
            if (p1 < end) {
                refit_points(p1, a1.in, a1.p.v, cs64(a1.p, a1.low), hy, (double)tau, stream_sums, o,
                             lane);
                if (p2 != p1 + stride) {
                    add_sums(a, stream_sums);
                    stream_sums = RefitSums();
                }
            }
            a0 = b0;
            a1 = b1;
            p0 = p2;
            p1 = p3;
        }
        add_sums(a, stream_sums);
    }
    if (shared) {
        __syncthreads();  // sh may lie where other LDS was read until now
        if (!kMore || wave < waves) {
            sh.sum[wave][0][lane] = a.scc;
            sh.sum[wave][1][lane] = a.scs;
            sh.sum[wave][2][lane] = a.sss;
            sh.sum[wave][3][lane] = a.scv;
            sh.sum[wave][4][lane] = a.ssv;
            sh.cnt[wave][0][lane] = a.n_in;
            sh.cnt[wave][1][lane] = a.n_near;
        }
        __syncthreads();
        if (wave > 0) return;
        a = RefitSums();
#pragma unroll 1
        for (int w = 0; w < kRefitStreams; ++w) {
            RefitSums t;
#pragma unroll 1
            for (int q = w; q < waves; q += kRefitStreams) {
                t.scc += sh.sum[q][0][lane];
                t.scs += sh.sum[q][1][lane];
                t.sss += sh.sum[q][2][lane];
                t.scv += sh.sum[q][3][lane];
                t.ssv += sh.sum[q][4][lane];
                t.n_in += sh.cnt[q][0][lane];
                t.n_near += sh.cnt[q][1][lane];
            }
            add_sums(a, t);
        }
    }
    wave_sum_all(a);
    if (lane == 0) write_refit(o, k, hbest, a.n_in, a.n_near, a.scc, a.scs, a.sss, a.scv, a.ssv);
}

// ---- single frame ---------------------------------------------------------

// Merges the workgroup's key into cluster j's and returns 1 in every lane of the calling
// wave when all `parts` of the cluster have done so, else 0.  The workgroups exchange
// nothing but the two words, both by atomic operations of the whole device: the merge has
// returned before the count is raised, so the last one's read sees every merge.  (A fence
// would also invalidate the XCD's L2: scoring of 4096 mixed clusters 146 us for 74.)
template <typename ClusterAt>
__device__ __forceinline__ uint32_t merge_part(const ClusterAt &at, int64_t j, unsigned long long key,
                                               uint32_t parts, int lane) {
    uint32_t last = 0;
    if (lane == 0) {
        const unsigned long long before = atomicMax(at.key(j), key);
        __builtin_amdgcn_s_waitcnt(0);
        last = at.arrive(j) == parts - 1 && before != ~0ull ? 1u : 0u;
    }
    return __builtin_amdgcn_readfirstlane(last);
}

// Cluster at planned position j of a single frame.
struct FrameClusterAt {
    const int32_t *off;
    int32_t *order;
    int64_t n_points;
    uint32_t key0, key1, cluster_base;
    int64_t point_base;
    unsigned long long *best_key;
    // The upper half of an entry counts the cluster's parts that are done, where the last
    // one refits it (there is an order for up to 65,536 clusters).
    __device__ int64_t index(int64_t j) const { return order != nullptr ? order[j] & 0xFFFF : j; }
    __device__ uint32_t arrive(int64_t j) const {
        return atomicAdd(reinterpret_cast<uint32_t *>(order) + j, 1u << 16) >> 16;
    }
    __device__ Span span(int64_t j) const {
        return cluster_span(off, index(j), n_points, point_base);
    }
    __device__ unsigned long long best(int64_t j) const { return best_key[index(j)]; }
    __device__ unsigned long long *key(int64_t j) const { return &best_key[index(j)]; }
    __device__ unsigned long long merged(int64_t j) const { return read_key(key(j)); }
    __device__ ClusterId id(int64_t j) const {
        ClusterId c;
        c.out = index(j);
        c.local = cluster_base + (uint32_t)c.out;
        c.key0 = key0;
        c.key1 = key1;
        return c;
    }
};

// refit_big (a workgroup has all hypotheses of a cluster, clusters are many): the
// workgroup refits its cluster itself from kRefitBigPoints on.  The points are still
// in the XCD's L2 and the work runs beside other clusters' scoring.  Smaller ones
// are cheaper a wave each (refit_planned): here they would hold a whole workgroup for
// the refit's chain of latencies.  4096 clusters of 8 to 4096 points, 1024
// hypotheses: score and refit 69.7 + 16.9 us apart, 73.8 + 10.9 us so (call 94.4 and
// 92.5 us); from 512 points on, 4096 clusters of 512 points take 97.4 us for 91.9.
// The batched kernel does not: its registers spill (256 frames 2369 to 2426 us).
//
// n_split (nullable; with refit_big): the first *n_split clusters are split between `parts`
// workgroups of `rounds` blocks (see kSplitPoints), which do not refit them, and each
// other cluster has one workgroup, behind them.
//
// Work item = (cluster, `rounds` blocks of 256 hypotheses).  Block i takes the
// item that keeps clusters in the planned order while all items of one cluster
// run on the same XCD (blocks are dealt to the 8 XCDs round-robin), sharing that
// XCD's L2 copy of the cluster's points.  Eight waves per SIMD: the scoring loop
// fits in 64 VGPRs.
template <int B>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(B == kLongBlock ? 4 : 8))) void score_kernel(
    const int32_t *__restrict__ off, int32_t *order, int64_t n_clusters,
    int64_t n_points, int32_t n_hyp, int32_t rounds, int32_t parts, uint32_t key0, uint32_t key1,
    uint32_t cluster_base, int64_t point_base, int32_t small_max, int64_t prune, Points pts,
    float tau, unsigned long long *__restrict__ best_key, Outputs o, bool refit_big,
    const int64_t *__restrict__ n_split, bool defer) {
    __shared__ ScoreShared<B> s;
    const uint32_t xcd = blockIdx.x % kXcds;
    const uint32_t r = blockIdx.x / kXcds;
    int64_t j = xcd + (int64_t)kXcds * (r / (uint32_t)parts);
    uint32_t part = r % (uint32_t)parts;
    const int64_t split = n_split != nullptr ? *n_split : 0;
    const bool whole = n_split != nullptr && blockIdx.x >= split * parts;  // not split
    if (whole) {
        j = blockIdx.x - split * (parts - 1);
        part = 0;
        rounds *= parts;
    }
    if (j >= n_clusters) return;
    const FrameClusterAt at = {off, order, n_points, key0, key1, cluster_base, point_base,
                               best_key};
    const int64_t k = at.index(j);
    const ClusterId id = at.id(j);
    const Span sp = at.span(j);
    const int most = rounds * B;
    const int64_t first = (int64_t)part * most;
    const int64_t left = n_hyp - first;
    const unsigned long long key = score_hypotheses<B, B == kLongBlock ? kPassRows : kFrameRows>(
        sp, id, first, left < most ? (int)left : most, n_hyp, pts, tau, kRowsMax, kSingleLanesMax,
        small_max, prune, false, defer, s, &best_key[k], o.hyp_counts);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (refit_big && (n_split == nullptr || whole) && sp.n >= kRefitBigPoints)
        refit_cluster(sp, id, key, pts, tau, o, wave, B / kWave, s.refit());
    else
        merge_key(&best_key[k], key, wave, threadIdx.x % kWave);
}

// Workgroup LDS of a refit kernel.
template <int B>
struct DeferredShared {
    float4 hyp[kScoreBlock / 2];
    uint32_t count[B / kScoreBlock][kScoreBlock];
    unsigned long long key[kScoreBlock / kWave];
    uint32_t last;
};

template <int B>
struct RefitSpace {
    static constexpr size_t kBytes = sizeof(RefitShared<B / kWave>);
    static_assert(sizeof(DeferredShared<B>) <= kBytes, "the larger");
    alignas(16) unsigned char bytes[kBytes];
    __device__ RefitShared<B / kWave> &refit() { return *reinterpret_cast<RefitShared<B / kWave> *>(bytes); }
    __device__ DeferredShared<B> &deferred() { return *reinterpret_cast<DeferredShared<B> *>(bytes); }
};

// Counts hypotheses [b 256, b 256 + 256) of a cluster in full: four waves with 64
// hypotheses each, or in a large workgroup four such groups with a quarter of the
// points each.  The best key, the same in every thread of the first four waves.
template <int B>
__device__ __forceinline__ unsigned long long count_block(Span sp, ClusterId id, int b, int32_t n_hyp,
                                                          const Points &pts, float tau, int wave,
                                                          DeferredShared<B> &sh) {
    constexpr int kGroups = B / kScoreBlock, kWaves = kScoreBlock / kWave;
    const int tid = threadIdx.x, lane = tid % kWave;
    const int64_t h = (int64_t)b * kScoreBlock + tid;
    float2 *hyp = reinterpret_cast<float2 *>(sh.hyp);
    if (wave < kWaves) {
        float2 own = make_float2(__builtin_nanf(""), __builtin_nanf(""));
        if (h < n_hyp) {
            const Hypothesis y = make_hypothesis(pts, sp, (uint32_t)h, id.local, id.key0, id.key1);
            own = make_float2((float)y.vx, (float)y.vy);
        }
        hyp[tid] = own;
    }
    __syncthreads();
    const int group = wave / kWaves, w = wave % kWaves;
    const int64_t rows = (sp.n + kWave - 1) / kWave;
    const int64_t r0 = rows * group / kGroups, r1 = rows * (group + 1) / kGroups;
    Span part;
    part.lo = sp.lo + r0 * kWave;
    part.n = (r1 * kWave < sp.n ? r1 * kWave : sp.n) - r0 * kWave;
    part.ok = true;
    sh.count[group][w * kWave + lane] = score_cluster<kPassRows, true>(
        pts, part, lane, sh.hyp + w * (kWave / 2), kWave, tau, kPassRows);
    __syncthreads();
    if (wave < kWaves) {
        uint32_t cnt = 0;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) cnt += sh.count[g][tid];
        const unsigned long long key = wave_best(__builtin_isnan(hyp[tid].x) ? 0u : cnt + 1u, (uint32_t)h);
        if (lane == 0) sh.key[wave] = key;
    }
    __syncthreads();
    return block_key<kScoreBlock>(sh.key);
}

// The deferred clusters (see score_pruned), counted in full in items of 256 hypotheses,
// dealt round the workgroups [n_clusters, gridDim.x) of a refit kernel in the planned
// order (largest first), a cluster's on one XCD.  A workgroup looks at 64 of its items
// at a time; one that ends the last item of a cluster refits it, so none waits for
// another.  These workgroups start when the others' refits are under way: a call without
// deferred clusters hardly sees them, as a launch of their own it would have
// (4096 mixed clusters 84 us of scoring for 75).
template <int B, typename ClusterAt>
__device__ __forceinline__ void refit_deferred(int64_t n_clusters, int32_t n_hyp,
                                               const ClusterAt &at, const Points &pts, float tau,
                                               const Outputs &o, int wave, RefitSpace<B> &space) {
    DeferredShared<B> &sh = space.deferred();
    const int lane = threadIdx.x % kWave;
    const uint32_t xcd = blockIdx.x % kXcds;
    const uint32_t step = (uint32_t)(gridDim.x - n_clusters) / kXcds;  // a multiple of kXcds
    const uint32_t blocks = ((uint32_t)n_hyp + kScoreBlock - 1) / kScoreBlock;
    const int64_t clusters = n_clusters > (int64_t)xcd ? (n_clusters - xcd + kXcds - 1) / kXcds : 0;
    const int64_t items = clusters * blocks;
    for (int64_t first = (blockIdx.x - n_clusters) / kXcds; first < items;
         first += (int64_t)step * kWave) {
        const int64_t mine = first + (int64_t)lane * step;
        const bool here = mine < items && at.best(xcd + kXcds * (mine / blocks)) >= kDeferred;
        for (uint64_t m = __builtin_amdgcn_ballot_w64(here); m != 0; m &= m - 1) {
            const int64_t item = first + (int64_t)__builtin_ctzll(m) * step;
            const int64_t j = xcd + kXcds * (item / blocks);
            const Span sp = at.span(j);
            const ClusterId id = at.id(j);
            const unsigned long long key =
                count_block<B>(sp, id, (int)(item % blocks), n_hyp, pts, tau, wave, sh);
            if (wave == 0) sh.last = merge_part(at, j, key | kDeferred, blocks, lane);
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(sh.last) != 0)
                refit_cluster(sp, id, at.merged(j) & ~kDeferred, pts, tau, o, wave, B / kWave,
                              space.refit());
            __syncthreads();
        }
    }
}

// Clusters that their scoring workgroups have refit: none, those of kRefitBigPoints
// points or more, or of these the ones that are not split.
enum RefitDone : int32_t { kNoneDone = 0, kBigDone = 1, kUnsplitDone = 2 };

// Refit of a frame's or batch's clusters over their planned (largest-first)
// positions, in one launch: workgroups [0, n_big) take the first n_big
// clusters (kRefitBigPoints or more, see there for frames of few), one each with
// all its waves; the following workgroups take the other clusters one per wave.  n_big is counted on the
// device by the ordering pass; without an order (n_big == nullptr) every
// cluster gets a workgroup.  The grid is an upper bound (one workgroup per
// cluster); surplus workgroups exit at once.  done: which of the
// big clusters were refit by their scoring workgroups.
//
// Behind them, where clusters may have been deferred: gridDim.x - n_clusters workgroups
// that count and refit those (refit_deferred).
template <int B, typename ClusterAt>
__device__ __forceinline__ void refit_planned(int64_t n_clusters, const int64_t *n_big,
                                              const ClusterAt &at, int32_t n_hyp, const Points &pts,
                                              float tau, const Outputs &o, RefitSpace<B> &space,
                                              RefitDone done) {
    constexpr int kWaves = B / kWave;
    RefitShared<kWaves> &sh = space.refit();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if constexpr (B == kLongBlock) {
        if (blockIdx.x >= n_clusters) {
            refit_deferred<B>(n_clusters, n_hyp, at, pts, tau, o, wave, space);
            return;
        }
    }
    const int64_t big = n_big != nullptr ? n_big[0] : n_clusters;
    int64_t b = blockIdx.x;
    if (done != kNoneDone) {
        const int64_t from = done == kBigDone ? 0 : n_big[1] < big ? n_big[1] : big;
        if (b >= from) b += big - from;
    }
    const bool all = b < big;  // the whole workgroup on one cluster
    const int64_t j = all ? b : big + (b - big) * kWaves + wave;
    if (j >= n_clusters) return;
    const unsigned long long best = at.best(j);
    if (B == kLongBlock && best >= kDeferred) return;
    refit_cluster(at.span(j), at.id(j), best, pts, tau, o, all ? wave : 0, all ? kWaves : 1, sh);
}

template <int B>
__global__ __launch_bounds__(B) void refit_kernel(
    const int32_t *__restrict__ off, int32_t *order, int64_t n_clusters,
    const int64_t *__restrict__ n_big, int64_t n_points, int32_t n_hyp, uint32_t key0, uint32_t key1,
    uint32_t cluster_base, int64_t point_base, Points pts, unsigned long long *best_key, float tau,
    Outputs o, RefitDone done) {
    __shared__ RefitSpace<B> s_refit;
    const FrameClusterAt at = {off, order, n_points, key0, key1, cluster_base, point_base,
                               best_key};
    refit_planned<B>(n_clusters, n_big, at, n_hyp, pts, tau, o, s_refit, done);
}

// Small frames (see use_cluster_path): one workgroup per cluster stages the
// cluster's own points, scores its hypotheses (at most 256) and refits, in a
// single launch.  The arithmetic is the three-kernel path's, so every output is
// the same; these frames are bound by launch latency, and one launch replaces
// three.  A workgroup reads back only points it staged itself, after a workgroup
// barrier (its waves share the compute unit's L1, which its own stores keep
// current; the staged points are written and read through one pointer, so no read
// of them goes through the scalar cache).
__global__ __launch_bounds__(kScoreBlock) __attribute__((amdgpu_waves_per_eu(8))) void cluster_kernel(
    const float *__restrict__ theta, const float *__restrict__ vd, const int32_t *__restrict__ off,
    int64_t n_points, int32_t n_hyp, uint32_t key0, uint32_t key1, uint32_t cluster_base,
    int64_t point_base, int32_t small_max, int64_t prune, float tau, Staging staged,
    Outputs o) {
    const Points pts = {staged.points, staged.low, theta};
    __shared__ ScoreShared<kScoreBlock> s;
    const int64_t k = blockIdx.x;
    const Span sp = cluster_span(off, k, n_points, point_base);
    for (int64_t p = sp.lo + threadIdx.x; p < sp.lo + sp.n; p += kScoreBlock)
        stage_point(theta, vd, p, staged);
    __syncthreads();
    ClusterId id;
    id.out = k;
    id.local = cluster_base + (uint32_t)k;
    id.key0 = key0;
    id.key1 = key1;
    const unsigned long long best =
        score_hypotheses<kScoreBlock, kPassRows>(sp, id, 0, n_hyp, n_hyp, pts, tau, kRowsMax,
                                                 kSingleLanesMax, small_max, prune, false, false, s,
                                                 nullptr, o.hyp_counts);
    refit_cluster(sp, id, best, pts, tau, o, __builtin_amdgcn_readfirstlane(threadIdx.x / kWave),
                  kScoreBlock / kWave, s.refit());
}

// ---- many frames in one launch sequence ----------------------------------
//
// The frames share one CSR: frame f owns clusters [frame_off[f], frame_off[f+1]).
// A cluster draws its hypotheses with its frame's seed and its index within
// the frame, so its result is bitwise the one a single-frame call gives.  The
// scoring kernel is persistent: a fixed grid drains device work queues of
// (cluster, up to 1024 hypotheses) items, clusters largest first.  There is one
// queue per XCD (its own 256-byte line): cluster j of the dispatch order
// belongs to queue j % 8, and workgroup b serves queue b % 8 first (workgroups
// are dispatched to the XCDs round-robin), so a cluster's blocks share one L2
// and no counter is hammered by the whole chip; a workgroup whose queue is
// empty takes items from the others.

struct Batch {
    const int32_t *frame_off;  // [n_frames + 1]
    const uint64_t *seeds;     // [n_frames], device
    int64_t n_frames;
};

// Register rows per pass for each cluster-size bucket: bucket 0 holds n < 64,
// bucket b holds n in [32 * 2^b, 64 * 2^b), the last bucket everything larger.
struct Tuning {
    int32_t rows[RV_TUNE_BUCKETS];
    int32_t fp16_min;   // clusters of at least this many points use the FP16 form; 0: none
    int32_t lanes_max;  // clusters of at most this many points score with lanes = hypotheses
    int32_t small_max;  // clusters of at most this many points take score_small
    int64_t prune;      // clusters of at least this many points count only possible winners
};

// Scoring form of a cluster (ItemDesc::form).
enum : uint8_t {
    kFormRows = 0,
    kFormFp16 = 1,
    kFormLanes = 2,
    kFormPruned = 3,
    kFormSmall = 4,
    kFormPrunedSmall = 5  // pruned; if that excludes too little, as kFormSmall
};

// Everything the scoring and refit workgroups need about one cluster, at its
// position in the dispatch order: one 32-byte load instead of a chain of
// dependent loads (order, offsets, frame, seed).
struct alignas(32) ItemDesc {
    int32_t lo, n;         // point span; n = 0 when the offsets are bad
    int32_t out;           // output index (the cluster's index in the batch)
    uint32_t local;        // counter word 1: index within its frame
    uint32_t key0, key1;   // Philox key: its frame's seed
    uint32_t done;         // parts of a deferred cluster's count that are done
    uint8_t ok;            // offsets valid
    uint8_t form;          // kFormRows etc.
    int16_t rows;          // register rows per pass for its size
};

constexpr int kQueueStride = 32;  // 64-bit counters: 256 bytes between queues

__device__ __forceinline__ int size_bucket(int64_t n) {
    int b = 0;
    while (b < RV_TUNE_BUCKETS - 1 && n >= ((int64_t)64 << b)) ++b;
    return b;
}

// Frame of cluster k: the last f with frame_off[f] <= k (binary search; stays
// inside [0, n_frames) whatever the offsets hold).
__device__ __forceinline__ int64_t frame_of_cluster(const int32_t *__restrict__ fo,
                                                    int64_t n_frames, int64_t k) {
    int64_t lo = 0, hi = n_frames;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) / 2;
        if (fo[mid] <= k)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

__device__ __forceinline__ Span desc_span(const ItemDesc &d) {
    Span sp;
    sp.lo = d.lo;
    sp.n = d.n;
    sp.ok = d.ok != 0;
    return sp;
}

__device__ __forceinline__ ClusterId desc_id(const ItemDesc &d) {
    ClusterId id;
    id.out = d.out;
    id.local = d.local;
    id.key0 = d.key0;
    id.key1 = d.key1;
    return id;
}

__device__ __forceinline__ int desc_lanes(const ItemDesc &d) {
    return d.form == kFormLanes ? kLaneTile : 0;
}

__device__ __forceinline__ int desc_small(const ItemDesc &d) {
    return d.form == kFormSmall ? kLaneTile : d.form == kFormPrunedSmall ? 1 : 0;
}

__device__ __forceinline__ int64_t desc_prune(const ItemDesc &d) {
    return d.form == kFormPruned || d.form == kFormPrunedSmall ? 0 : INT64_MAX;
}

// Runs body(cluster position, part) for every item this workgroup takes from the
// queues: cluster j of the dispatch order belongs to queue j % 8, `parts` items
// each; a workgroup serves its home queue (home = blockIdx.x % 8) first, then the
// others.  Its first item is fixed, number blockIdx.x / 8 of its home queue; the
// queue's counter gives out those behind the fixed ones, and a queue with none behind
// them is not asked: a batch that the grid holds at once runs without an atomic
// (one for the first item and one for each of the eight empty queues at the end, one
// after the other: 8 frames of 100 clusters 51.9 and 34.8 us, 3 of 700 78.4 and 75.4
// us, 64 of 700 423 and 419 us).  Looking at all eight counters with one load instead
// was slower than the atomics (64 frames 434 us).
// The body is called by the whole workgroup and may hold barriers (see
// batch_score_kernel).
template <typename Body>
__device__ __forceinline__ void for_each_item(unsigned long long *__restrict__ queues,
                                              int64_t n_clusters, int32_t parts, uint32_t home,
                                              int wave, int lane, unsigned long long &s_item,
                                              const Body &body) {
    const auto total = [&](uint32_t q) {
        const int64_t clusters_q = n_clusters > (int64_t)q ? (n_clusters - q + kXcds - 1) / kXcds : 0;
        return (unsigned long long)clusters_q * (uint64_t)parts;
    };
    uint32_t step = 0, q = home;
    unsigned long long item = blockIdx.x / kXcds;
    bool found = item < total(home);
    for (;;) {  // one copy of the body: a second one costs its instruction fetches
        if (found) {
            const unsigned long long at = item / (uint64_t)parts;
            body((int64_t)q + (int64_t)kXcds * (int64_t)at, (int)(item - at * (uint64_t)parts));
        }
        found = false;
        while (!found && step < kXcds) {
            q = (home + step) % kXcds;
            const unsigned long long n = total(q);
            const unsigned long long fixed = gridDim.x > q ? (gridDim.x - q + kXcds - 1) / kXcds : 0;
            if (fixed < n) {
                if (wave == 0) {
                    unsigned long long got = 0;
                    if (lane == 0) got = atomicAdd(&queues[q * kQueueStride], 1ull);
                    s_item = uniform_u64(got) + fixed;  // the same value from every lane of wave 0
                }
                __syncthreads();
                item = uniform_u64(s_item);
                __syncthreads();
                found = item < n;
            }
            step += found ? 0 : 1;
        }
        if (!found) break;
    }
}

// Descriptor of cluster k of frame f.
__device__ __forceinline__ void write_desc(int64_t k, const Span &sp, int64_t f, const Batch &bt,
                                           const Tuning &tune, ItemDesc &at) {
    const uint64_t seed = bt.seeds[f];
    ItemDesc d;
    d.lo = (int32_t)sp.lo;
    d.n = (int32_t)sp.n;
    d.out = (int32_t)k;
    d.local = (uint32_t)(k - bt.frame_off[f]);
    d.key0 = (uint32_t)(seed & 0xFFFFFFFFu);
    d.key1 = (uint32_t)(seed >> 32);
    d.done = 0;
    d.ok = sp.ok ? 1 : 0;
    d.rows = (int16_t)tune.rows[size_bucket(sp.n)];
    d.form = kFormRows;
    if (sp.n >= 2 && sp.n <= tune.small_max)
        d.form = kFormSmall;
    else if (sp.ok && sp.n >= 2 && sp.n <= tune.lanes_max)
        d.form = kFormLanes;
    else if (tune.fp16_min > 0 && sp.ok && sp.n >= 2 && sp.n >= tune.fp16_min)
        d.form = kFormFp16;
    else if (sp.n >= tune.prune)
        d.form = tune.small_max > 0 && sp.n <= kLaneTile ? kFormPrunedSmall : kFormPruned;
    at = d;
}

// Places taken so far of size class c in the dispatch order: a counter in the
// second half of the queues' 256-byte lines.
__device__ __forceinline__ uint32_t *class_cursor(unsigned long long *queues, int c) {
    static_assert(kSizeClasses == 16 * kXcds && kQueueStride == 32, "16 classes a queue");
    return reinterpret_cast<uint32_t *>(queues + (c / 16) * kQueueStride + kQueueStride / 2) + c % 16;
}

// Clears the size-class histogram, the classes' cursors and the work queues.
__global__ __launch_bounds__(kSizeClasses) void batch_init_kernel(
    uint32_t *__restrict__ hist, unsigned long long *__restrict__ queues) {
    hist[threadIdx.x] = 0;
    *class_cursor(queues, threadIdx.x) = 0;
    if (threadIdx.x < kXcds) queues[threadIdx.x * kQueueStride] = 0;
}

// One thread per point: staging as in prep_kernel.  One thread per cluster:
// clear its best key and count it in its size class (per-block LDS histogram,
// one global atomic per class and block).
__global__ __launch_bounds__(kPrepBlock) void batch_prep_kernel(
    const float *__restrict__ theta, const float *__restrict__ vd, int64_t n_points,
    Staging staged, uint32_t *__restrict__ bits, int64_t n_words,
    const int32_t *__restrict__ off, int64_t n_clusters, unsigned long long *__restrict__ best_key, uint32_t *__restrict__ hist) {
    __shared__ uint32_t local[kSizeClasses];
    for (int c = threadIdx.x; c < kSizeClasses; c += kPrepBlock) local[c] = 0;
    __syncthreads();
    const int64_t p = (int64_t)blockIdx.x * kPrepBlock + threadIdx.x;
    if (p < n_points) stage_point(theta, vd, p, staged);
    if (bits != nullptr && p < n_words) bits[p] = 0u;
    if (p < n_clusters) {
        best_key[p] = 0;
        atomicAdd(&local[size_class(cluster_span(off, p, n_points).n)], 1u);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < kSizeClasses; c += kPrepBlock)
        if (local[c] != 0) atomicAdd(&hist[c], local[c]);
}

// Batches of at most kPlanBatch clusters and kPlanFrames frames: the first workgroup
// orders them and writes their descriptors beside the staging of the others, as for
// a single frame, instead of two launches around it: one frame of 700 clusters of 8 to
// 1024 points 53.7 and 48.0 us, 64 clusters of 65,536 points 178.7 and 171.2 us.  At
// 2800 clusters in four frames the one workgroup is the longer way (82.3 and 85.6 us).
constexpr int kPlanBatchEach = 4;  // clusters a thread
constexpr int64_t kPlanBatch = kPlanBatchEach * kPrepBlock;
constexpr int64_t kPlanFrames = 1024;

bool plan_in_prep(int64_t n_clusters, int64_t n_frames) {
    return n_clusters <= kPlanBatch && n_frames <= kPlanFrames;
}

__device__ void plan_batch(const int32_t *__restrict__ off, int64_t n_clusters, int64_t n_points,
                           Batch bt, const Tuning &tune, unsigned long long *__restrict__ queues,
                           int64_t *__restrict__ n_big, ItemDesc *__restrict__ desc) {
    __shared__ uint32_t count[kSizeClasses];
    __shared__ uint32_t start[kSizeClasses];
    __shared__ int32_t frame_off[kPlanFrames + 1];
    for (int c = threadIdx.x; c < kSizeClasses; c += kPrepBlock) count[c] = 0;
    for (int f = threadIdx.x; f <= (int)bt.n_frames; f += kPrepBlock) frame_off[f] = bt.frame_off[f];
    if (threadIdx.x < kXcds) queues[threadIdx.x * kQueueStride] = 0;
    __syncthreads();
    int cls[kPlanBatchEach];
#pragma unroll
    for (int u = 0; u < kPlanBatchEach; ++u) {
        const int64_t k = threadIdx.x + (int64_t)u * kPrepBlock;
        cls[u] = k < n_clusters ? size_class(cluster_span(off, k, n_points).n) : -1;
    }
#pragma unroll
    for (int u = 0; u < kPlanBatchEach; ++u)
        if (cls[u] >= 0) atomicAdd(&count[cls[u]], 1u);
    __syncthreads();
    plan_scan(count, start, refit_big_class(n_clusters), 0, n_big);
    __syncthreads();
    for (int64_t k = threadIdx.x; k < n_clusters; k += kPrepBlock) {
        const Span sp = cluster_span(off, k, n_points);
        const uint32_t pos = atomicAdd(&start[size_class(sp.n)], 1u);
        write_desc(k, sp, frame_of_cluster(frame_off, bt.n_frames, k), bt, tune, desc[pos]);
    }
}

__global__ __launch_bounds__(kPrepBlock) void batch_plan_prep_kernel(
    const float *__restrict__ theta, const float *__restrict__ vd, int64_t n_points,
    Staging staged, uint32_t *__restrict__ bits, int64_t n_words,
    const int32_t *__restrict__ off, int64_t n_clusters, Batch bt, Tuning tune,
    unsigned long long *__restrict__ best_key, unsigned long long *__restrict__ queues,
    int64_t *__restrict__ n_big, ItemDesc *__restrict__ desc) {
    if (blockIdx.x == 0) {
        plan_batch(off, n_clusters, n_points, bt, tune, queues, n_big, desc);
        return;
    }
    const int64_t p = (int64_t)(blockIdx.x - 1) * kPrepBlock + threadIdx.x;
    if (p < n_points) stage_point(theta, vd, p, staged);
    if (bits != nullptr && p < n_words) bits[p] = 0u;
    if (p < n_clusters) best_key[p] = 0;
}

// Places every cluster in the dispatch order (one global atomic per class and
// block reserves a range, LDS atomics rank the block's clusters inside it) and
// writes its descriptor there.  Every block scans the histogram for the classes'
// starts itself (a launch of one wave for it: 1.5 us more of every batch).
__global__ __launch_bounds__(kPrepBlock) void batch_scatter_kernel(
    const int32_t *__restrict__ off, int64_t n_clusters, int64_t n_points, Batch bt, Tuning tune,
    const uint32_t *__restrict__ hist, unsigned long long *__restrict__ queues,
    int64_t *__restrict__ n_big, ItemDesc *__restrict__ desc) {
    __shared__ uint32_t total[kSizeClasses];
    __shared__ uint32_t start[kSizeClasses];
    __shared__ uint32_t count[kSizeClasses];
    __shared__ uint32_t base[kSizeClasses];
    __shared__ int64_t s_big[2];
    for (int c = threadIdx.x; c < kSizeClasses; c += kPrepBlock) {
        count[c] = 0;
        total[c] = hist[c];
    }
    __syncthreads();
    plan_scan(total, start, refit_big_class(n_clusters), 0, s_big);
    const int64_t k = (int64_t)blockIdx.x * kPrepBlock + threadIdx.x;
    int cls = -1;
    uint32_t rank = 0;
    Span sp;
    if (k < n_clusters) {
        sp = cluster_span(off, k, n_points);
        cls = size_class(sp.n);
        rank = atomicAdd(&count[cls], 1u);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < kSizeClasses; c += kPrepBlock)
        base[c] = count[c] != 0 ? start[c] + atomicAdd(class_cursor(queues, c), count[c]) : 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) n_big[0] = s_big[0];
    __syncthreads();
    if (cls < 0) return;
    write_desc(k, sp, frame_of_cluster(bt.frame_off, bt.n_frames, k), bt, tune, desc[base[cls] + rank]);
}

// Persistent scoring over the per-XCD queues (see above).  Every branch that
// leads to or around a barrier in the item loop is taken on a wave-uniform
// value (wave index, item read back with readfirstlane): with a per-lane guard
// such as threadIdx.x == 0 the compiler may thread that guard across the
// loop's back edge into a lane-masked inner loop that lane 0 leaves to fetch
// the next item while lanes 1..63 wait on the old one.  The float32-only
// instantiation runs eight waves per SIMD (a few reloads of loop state per pass
// of rows, measured 1-2 % faster than seven waves without them); kFp16: the
// instantiation that also runs FP16-form items (launched only when the tuning
// enables that form, so that the float32-only kernel keeps its own register
// allocation), at seven waves per SIMD.  The large workgroups of long clusters come
// one to a CU, so they have the registers of four waves per SIMD.
template <bool kFp16, int B>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(B == kLongBlock ? 4 : kFp16 ? 7 : 8))) void batch_score_kernel(
    const ItemDesc *__restrict__ desc, int64_t n_clusters, int32_t n_hyp,
    int32_t rounds, int32_t parts, int64_t prune, bool defer, Points pts, float tau,
    unsigned long long *__restrict__ queues, unsigned long long *__restrict__ best_key,
    int32_t *__restrict__ hyp_counts) {
    __shared__ ScoreShared<B> s;
    __shared__ unsigned long long s_item;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const uint32_t home = blockIdx.x % kXcds;
    for_each_item(queues, n_clusters, parts, home, wave, lane, s_item, [&](int64_t j, int part) {
        const ItemDesc d = desc[j];
        const int most = rounds * B;
        const int64_t first = (int64_t)part * most;
        const int64_t left = n_hyp - first;
        const int nh = left < most ? (int)left : most;
        const bool half = kFp16 && d.form == kFormFp16 && d.n >= prune;
        if constexpr (kFp16 && B == kScoreBlock) {
            if (d.form == kFormFp16 && !half) {
                const int b0 = part * rounds;
                for (int b = b0; b < b0 + (nh + kScoreBlock - 1) / kScoreBlock; ++b) {
                    score_block_fp16(desc_span(d), desc_id(d), b, n_hyp, pts, tau, d.rows, s.fp16(),
                                     best_key, hyp_counts);
                    __syncthreads();
                }
                return;
            }
        }
        const unsigned long long key = score_hypotheses<B, kPassRows, kFp16>(
            desc_span(d), desc_id(d), first, nh, n_hyp, pts, tau, d.rows, desc_lanes(d),
            desc_small(d), half ? 0 : desc_prune(d), half, defer, s,
            &best_key[d.out], hyp_counts);
        merge_key(&best_key[d.out], key, wave, lane);
    });
}

// Cluster at dispatch position j of a batch (its descriptor).
struct BatchClusterAt {
    ItemDesc *desc;
    unsigned long long *best_key;
    __device__ Span span(int64_t j) const { return desc_span(desc[j]); }
    __device__ ClusterId id(int64_t j) const { return desc_id(desc[j]); }
    __device__ unsigned long long best(int64_t j) const { return best_key[desc[j].out]; }
    __device__ unsigned long long *key(int64_t j) const { return &best_key[desc[j].out]; }
    __device__ unsigned long long merged(int64_t j) const { return read_key(key(j)); }
    __device__ uint32_t arrive(int64_t j) const { return atomicAdd(&desc[j].done, 1u); }
};

template <int B>
__global__ __launch_bounds__(B) void batch_refit_kernel(
    ItemDesc *desc, int64_t n_clusters, const int64_t *__restrict__ n_big, int32_t n_hyp, Points pts,
    unsigned long long *best_key, float tau, Outputs o) {
    __shared__ RefitSpace<B> s_refit;
    const BatchClusterAt at = {desc, best_key};
    refit_planned<B>(n_clusters, n_big, at, n_hyp, pts, tau, o, s_refit, kNoneDone);
}

__global__ __launch_bounds__(kPrepBlock) void philox_kernel(const uint32_t *__restrict__ ctr,
                                                        const uint32_t *__restrict__ key,
                                                        uint32_t *__restrict__ out,
                                                        int64_t n) {
    const int64_t t = (int64_t)blockIdx.x * kPrepBlock + threadIdx.x;
    if (t >= n) return;
    const uint4 r = philox4x32_10(
        make_uint4(ctr[4 * t], ctr[4 * t + 1], ctr[4 * t + 2], ctr[4 * t + 3]), key[2 * t],
        key[2 * t + 1]);
    out[4 * t] = r.x;
    out[4 * t + 1] = r.y;
    out[4 * t + 2] = r.z;
    out[4 * t + 3] = r.w;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

using rv_internal::fail;
using rv_internal::g_error;
using rv_internal::g_free;
using rv_internal::g_pending;
using rv_internal::g_timing;
using rv_internal::g_timing_mutex;
using rv_internal::keep_timed_call;
using rv_internal::kStages;
using rv_internal::take_timed_call;
using rv_internal::TimedCall;

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Layout {
    size_t staged, low, order, best_key, n_big, total;
};

// The points' 12-byte records, with the room of two aligned arrays of 8 and 4 bytes
// a point: rv_workspace_bytes has always answered with that size, and callers keep
// workspaces by it.
size_t staged_bytes(size_t n_points) {
    static_assert(sizeof(StagedPoint) == 3 * sizeof(float), "12-byte records");
    return align_up(align_up(n_points * 2 * sizeof(float)) + n_points * sizeof(float));
}

Layout make_layout(int64_t n_clusters, int64_t n_points) {
    Layout L;
    const size_t np = (size_t)n_points;
    size_t at = 0;
    L.staged = at; at += staged_bytes(np);
    L.low = at; at = align_up(at + np * sizeof(StagedLow));
    L.order = at; at = align_up(at + (size_t)n_clusters * sizeof(int32_t));
    L.best_key = at; at = align_up(at + (size_t)n_clusters * sizeof(unsigned long long));
    L.n_big = at; at = align_up(at + 2 * sizeof(int64_t));
    L.total = at;
    return L;
}

// Stage timing: events recorded around each kernel of each call.


struct BatchLayout {
    size_t staged, low, desc, best_key, hist, queues, n_big, total;
};

BatchLayout make_batch_layout(int64_t n_clusters, int64_t n_points) {
    BatchLayout L;
    const size_t np = (size_t)n_points, nc = (size_t)n_clusters;
    size_t at = 0;
    L.staged = at; at += staged_bytes(np);
    L.low = at; at = align_up(at + np * sizeof(StagedLow));
    L.desc = at; at = align_up(at + nc * sizeof(ItemDesc));
    L.best_key = at; at = align_up(at + nc * sizeof(unsigned long long));
    L.hist = at; at = align_up(at + kSizeClasses * sizeof(uint32_t));
    L.queues = at; at = align_up(at + kXcds * kQueueStride * sizeof(unsigned long long));
    L.n_big = at; at = align_up(at + 2 * sizeof(int64_t));
    L.total = at;
    return L;
}

struct BatchArgs {
    const float *theta, *vd;
    const int32_t *off, *frame_off;
    const uint64_t *seeds;
    int64_t n_frames, n_clusters, n_points;
    int32_t n_hyp;
    float tau;
    Outputs o;
    rv_tuning_t tuning;
    void *workspace;
    size_t workspace_bytes;
};

int check_batch(const BatchArgs &a) {
    if (a.n_frames < 1 || a.n_frames > (int64_t)INT32_MAX)
        return fail(RV_ERR_INVALID_ARG, "n_frames must be in [1, 2^31 - 1]");
    if (a.n_clusters < 0 || a.n_clusters > (int64_t)INT32_MAX)
        return fail(RV_ERR_INVALID_ARG, "n_clusters must be in [0, 2^31 - 1]");
    if (a.n_points < 0 || a.n_points > INT32_MAX)
        return fail(RV_ERR_INVALID_ARG, "n_points must be in [0, 2^31 - 1]");
    if (a.n_hyp < 1 || a.n_hyp > RV_MAX_HYP)
        return fail(RV_ERR_INVALID_ARG, "n_hyp must be in [1, %d]", RV_MAX_HYP);
    if (!(a.tau > 0.0f) || !isfinite(a.tau))
        return fail(RV_ERR_INVALID_ARG, "tau must be finite and > 0");
    if (a.off == nullptr || a.frame_off == nullptr || a.seeds == nullptr)
        return fail(RV_ERR_INVALID_ARG, "cluster_offsets, frame_offsets or seeds is NULL");
    if (a.n_points > 0 && (a.theta == nullptr || a.vd == nullptr))
        return fail(RV_ERR_INVALID_ARG, "theta or vd is NULL");
    if (a.n_clusters > 0 && (a.o.vx == nullptr || a.o.vy == nullptr || a.o.heading == nullptr ||
                             a.o.n_inliers == nullptr || a.o.status == nullptr))
        return fail(RV_ERR_INVALID_ARG, "a required output is NULL");
    for (int b = 0; b < RV_TUNE_BUCKETS; ++b)
        if (a.tuning.rows_max[b] < 1 || a.tuning.rows_max[b] > kRowsMax)
            return fail(RV_ERR_INVALID_ARG, "tuning.rows_max must be in [1, %d]", kRowsMax);
    if (a.tuning.blocks_per_cu < 0 || a.tuning.blocks_per_cu > 64)
        return fail(RV_ERR_INVALID_ARG, "tuning.blocks_per_cu must be in [0, 64]");
    if (a.tuning.fp16_min_points < 0)
        return fail(RV_ERR_INVALID_ARG, "tuning.fp16_min_points must be >= 0");
    if (a.tuning.lanes_max_points < 0 || a.tuning.lanes_max_points > kLaneTile)
        return fail(RV_ERR_INVALID_ARG, "tuning.lanes_max_points must be in [0, %d]", kLaneTile);
    const BatchLayout L = make_batch_layout(a.n_clusters, a.n_points);
    if (a.workspace == nullptr || a.workspace_bytes < L.total)
        return fail(RV_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", L.total,
                    a.workspace == nullptr ? (size_t)0 : a.workspace_bytes);
    if (((uintptr_t)a.workspace % kAlign) != 0)
        return fail(RV_ERR_WORKSPACE, "workspace must be %zu-byte aligned", kAlign);
    return RV_OK;
}

int64_t blocks_of(int32_t n_hyp) { return ((int64_t)n_hyp + kScoreBlock - 1) / kScoreBlock; }

// Compute units of the current device, queried once per device (a launch that
// is being captured into a graph only reads the cache, filled by the caller's
// earlier call).
int device_cus() {
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    int cus = cache[dev].load(std::memory_order_relaxed);
    if (cus > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    cache[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

// Hypotheses per scoring workgroup, in blocks of 256 (at most kPruneHyp).  A
// large cluster's table is made once per workgroup, so as many as leave 2048
// workgroups (eight per compute unit): scoring stage with 1, 2 and 4 at 1024
// hypotheses: 4096 mixed clusters 116, 88 and 83 us; 1024 clusters of 2048 points
// 68, 55 and 68 us; 512 of 4096 points 56, 66 and 90 us.
int32_t score_rounds(int64_t n_clusters, int64_t blocks_per_cluster) {
    int32_t rounds = 1;
    while (rounds < kPruneHyp / kScoreBlock && rounds < blocks_per_cluster &&
           n_clusters * ((blocks_per_cluster + 2 * rounds - 1) / (2 * rounds)) >= 2048)
        rounds *= 2;
    return rounds;
}

// Smallest cluster that counts only possible winners: none when the caller asks
// for every hypothesis's count, or tau is so extreme that the residual bins'
// scale leaves the normal range.
bool ordinary_tau(float tau) { return tau > 1e-15f && tau < 1e15f; }

int64_t prune_from(int32_t rounds, float tau, const int32_t *hyp_counts) {
    return hyp_counts != nullptr || !ordinary_tau(tau) ? INT64_MAX : prune_min(rounds);
}

// Largest cluster that takes score_small; lanes_max: what the tuning lets take
// lanes = hypotheses (0: none).  Where a table pays (prune_min) that takes over:
// 32,768 clusters at 512 hypotheses, scoring stage this way 129, 161, 195 us at 64,
// 96 and 128 points (198, 245 and 256 us with lanes = points above 64 and one
// hypothesis per thread below), with a table 236 and 241 us at 128 and 192.  With one
// block per workgroup a broadcast serves one hypothesis and LDS sets the rate, yet
// nearly as far as the tile goes it is the shorter chain (call this way and with lanes =
// points: 4096 clusters of 210 points at 256 hypotheses 54.1 and 59.5 us, 1000 of 230 points
// at 512 28.0 and 30.7, 64 of 230 points 18.6 and 18.5; of 256 points 58.7 and 63.7,
// 29.3 and 30.8, but 18.4 and 17.4).
constexpr int32_t kSmallAlone = 240;

int32_t small_to(int32_t rounds, float tau, int32_t lanes_max) {
    if (lanes_max == 0 || !ordinary_tau(tau)) return 0;
    const int32_t most = rounds == 1 ? kSmallAlone : prune_min(rounds) - 1;
    return most > lanes_max ? most : lanes_max;
}

// Frames small enough that launch latency dominates take one launch
// (cluster_kernel): at most 256 hypotheses, at most 65,536 points (each workgroup
// stages its own cluster) and no frame-wide inlier mask (its words are shared by
// neighbouring clusters and are cleared by the staging kernel).
constexpr int64_t kSmallFrameMaxPoints = 1 << 16;
constexpr int64_t kSmallFrameMaxClusters = 1 << 16;

bool use_cluster_path(int64_t n_clusters, int64_t n_points, int32_t n_hyp,
                      const uint32_t *inlier_bits) {
    return inlier_bits == nullptr && n_hyp <= kScoreBlock && n_points <= kSmallFrameMaxPoints &&
           n_clusters <= kSmallFrameMaxClusters;
}

// Workgroups behind a refit kernel's own that count deferred clusters (a multiple of
// kXcds), and the most scoring workgroups of a call that defers: with a workgroup for
// every second compute unit, spreading a cluster over the chip still makes up for
// counting it twice in part (100 clusters of 8192 points, 90 % outliers: call 238 us
// counted in place, 142 us deferred; 200 clusters 206 and 262 us).
constexpr int kDeferredBlocks = 256;
constexpr int64_t kDeferItems = 128;

// Split of a call's scoring: workgroups of `block` threads, each with `rounds` blocks
// of hypotheses of a cluster, `parts` of them per cluster; the pruned form's smallest
// and score_small's largest cluster.
struct ScorePlan {
    int32_t block, rounds, parts, small_max;
    int64_t prune;
    bool defer;
};

// Few and long clusters (the mean length is what the host knows; the choice is one
// for speed alone) are scored by workgroups of 1024 threads with up to 1024 hypotheses
// each and refit by such.  In the small workgroups every 256 hypotheses of a cluster
// sweep all its points for their own table: 64 clusters of 65,536 points at 4096
// hypotheses, 16 workgroups each, score in 270 us and refit in 57 us, 4 and 1 large
// ones in 105 and 29 us (call 378 and 180 us, in the FP16 form 460 and 201 us).
// The line: scoring of 64 clusters at 1024 hypotheses 44.7 and 35.3 us at 8192 points,
// 28.0 and 28.8 us at 4096.  Beyond a workgroup per CU a large one's share is too
// coarse (320 x 8192 points at 300 hypotheses 53 and 65 us) unless it takes the place
// of four and the clusters are twice as long (512 x 16,384 points at 1024 hypotheses 153
// and 114 us, 90 % outliers 641 and 730; 300 x 8192 points 67 and 68 us, and with 90 %
// outliers 238 and 368).
constexpr int64_t kLongPoints = 8192;
constexpr int64_t kLongClusters = 256;

bool long_clusters(int64_t n_clusters, int64_t n_points) {
    return n_clusters > 0 && n_points / n_clusters >= kLongPoints;
}

ScorePlan plan_score(int64_t n_clusters, int64_t n_points, int32_t n_hyp, float tau,
                     const int32_t *hyp_counts, int32_t lanes_max, int32_t fp16_min) {
    ScorePlan p;
    p.block = kScoreBlock;
    // A full count has little to share between blocks and wants the finer split (frame
    // of 4096 clusters of 8 to 4096 points with hyp_counts: 312 us with four blocks per workgroup, 244 us with one).
    const bool pruned = prune_from(1, tau, hyp_counts) != INT64_MAX;
    p.rounds = pruned ? score_rounds(n_clusters, blocks_of(n_hyp)) : 1;
    const auto parts = [n_hyp](int64_t each) { return (int32_t)((n_hyp + each - 1) / each); };
    p.parts = parts(kScoreBlock * p.rounds);
    int32_t blocks = p.rounds;  // of 256 hypotheses, per workgroup
    // The large workgroups have no FP16 form of a full count: only where every
    // cluster of that form is pruned.
    constexpr int32_t kLongBlocks = kLongBlock / kScoreBlock;
    if (long_clusters(n_clusters, n_points) &&
        (n_clusters <= kLongClusters || (p.parts >= 4 * parts(kLongBlock) &&
                                         n_points / n_clusters >= 2 * kLongPoints)) &&
        pruned && (fp16_min <= 0 || fp16_min >= prune_min(kLongBlocks))) {
        p.block = kLongBlock;
        p.rounds = 1;
        p.parts = parts(kLongBlock);
        blocks = kLongBlocks;
    }
    p.prune = prune_from(blocks, tau, hyp_counts);
    p.small_max = small_to(blocks, tau, lanes_max);
    if (fp16_min > 0 && p.small_max >= fp16_min) p.small_max = fp16_min - 1;
    p.defer = p.block == kLongBlock && n_clusters * p.parts <= kDeferItems;
    return p;
}

ScorePlan batch_plan(const BatchArgs &a) {
    return plan_score(a.n_clusters, a.n_points, a.n_hyp, a.tau, a.o.hyp_counts,
                      a.tuning.lanes_max_points, a.tuning.fp16_min_points);
}

using BatchScore = void (*)(const ItemDesc *, int64_t, int32_t, int32_t, int32_t, int64_t, bool, Points,
                            float, unsigned long long *, unsigned long long *, int32_t *);
BatchScore batch_score(bool fp16, int32_t block) {
    if (block == kLongBlock)
        return fp16 ? batch_score_kernel<true, kLongBlock> : batch_score_kernel<false, kLongBlock>;
    return fp16 ? batch_score_kernel<true, kScoreBlock> : batch_score_kernel<false, kScoreBlock>;
}

// The refit kernel over planned positions; n_big (device, nullable) is the
// ordering pass's count of big clusters.
void launch_refit(bool batch, const int32_t *off, int32_t *order, ItemDesc *desc,
                  int64_t n_clusters, const int64_t *n_big, int64_t n_points, int32_t n_hyp,
                  uint32_t key0, uint32_t key1, uint32_t cluster_base, int64_t point_base,
                  const Points &pts, unsigned long long *best_key, float tau, const Outputs &o,
                  RefitDone done, bool large, bool defer, hipStream_t st) {
    const dim3 block(large ? kLongBlock : kRefitBlock);
    const dim3 grid((unsigned)(n_clusters + (defer ? kDeferredBlocks : 0)));
    if (batch)
        hipLaunchKernelGGL(large ? batch_refit_kernel<kLongBlock> : batch_refit_kernel<kRefitBlock>,
                           grid, block, 0, st, desc, n_clusters, n_big, n_hyp, pts, best_key, tau, o);
    else
        hipLaunchKernelGGL(large ? refit_kernel<kLongBlock> : refit_kernel<kRefitBlock>,
                           grid, block, 0, st, off, order, n_clusters, n_big, n_points, n_hyp, key0,
                           key1, cluster_base, point_base, pts, best_key, tau, o, done);
}

// Persistent grid of the batched scoring kernel on the current device.
int persistent_blocks(const BatchArgs &a, unsigned *grid) {
    *grid = 1;
    if (a.n_clusters == 0) return RV_OK;
    int fit = 0;
    const int cus = device_cus();
    const ScorePlan plan = batch_plan(a);
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &fit, batch_score(a.tuning.fp16_min_points > 0, plan.block), plan.block, 0);
    if (cus <= 0 || e != hipSuccess)
        return fail(RV_ERR_HIP, "device query failed");
    const int asked = a.tuning.blocks_per_cu;
    int per_cu = asked > 0 && asked < fit ? asked : fit;
    if (per_cu < 1) per_cu = 1;
    // As many for every queue as the longest has items (see for_each_item).
    const int64_t items = (a.n_clusters + kXcds - 1) / kXcds * kXcds * plan.parts;
    int64_t g = (int64_t)cus * per_cu;
    if (g > items) g = items;
    *grid = (unsigned)(g > 0 ? g : 1);
    return RV_OK;
}

// The launch sequence of the batched form (argument checks and the persistent
// grid size done by the caller, so that no device query falls inside a capture).
int launch_batch(const BatchArgs &a, unsigned grid, hipStream_t st, bool allow_timing) {
    if (a.n_clusters == 0) return RV_OK;
    const BatchLayout L = make_batch_layout(a.n_clusters, a.n_points);
    char *ws = (char *)a.workspace;
    const Staging staged = {(StagedPoint *)(ws + L.staged), (StagedLow *)(ws + L.low)};
    ItemDesc *desc = (ItemDesc *)(ws + L.desc);
    unsigned long long *best_key = (unsigned long long *)(ws + L.best_key);
    uint32_t *hist = (uint32_t *)(ws + L.hist);
    unsigned long long *queues = (unsigned long long *)(ws + L.queues);
    int64_t *n_big = (int64_t *)(ws + L.n_big);
    Points pts;
    pts.staged = staged.points;
    pts.low = staged.low;
    pts.theta = a.theta;
    Batch bt;
    bt.frame_off = a.frame_off;
    bt.seeds = a.seeds;
    bt.n_frames = a.n_frames;
    Tuning tune;
    for (int b = 0; b < RV_TUNE_BUCKETS; ++b) tune.rows[b] = a.tuning.rows_max[b];
    tune.fp16_min = a.tuning.fp16_min_points;
    tune.lanes_max = a.tuning.lanes_max_points;
    const ScorePlan plan = batch_plan(a);
    tune.prune = plan.prune;
    tune.small_max = plan.small_max;
    const int64_t n_words = a.o.bits != nullptr ? (a.n_points + 31) / 32 : 0;
    int64_t prep_items = a.n_points > n_words ? a.n_points : n_words;
    prep_items = prep_items > a.n_clusters ? prep_items : a.n_clusters;

    TimedCall tc;
    const bool timed = allow_timing && take_timed_call(tc);
    if (timed) (void)hipEventRecord(tc.ev[0], st);
    const unsigned prep_blocks = (unsigned)((prep_items + kPrepBlock - 1) / kPrepBlock);
    if (plan_in_prep(a.n_clusters, a.n_frames)) {
        hipLaunchKernelGGL(batch_plan_prep_kernel, dim3(prep_blocks + 1), dim3(kPrepBlock), 0, st,
                           a.theta, a.vd, a.n_points, staged, a.o.bits, n_words, a.off,
                           a.n_clusters, bt, tune, best_key, queues, n_big, desc);
    } else {
        hipLaunchKernelGGL(batch_init_kernel, dim3(1), dim3(kSizeClasses), 0, st, hist, queues);
        hipLaunchKernelGGL(batch_prep_kernel, dim3(prep_blocks), dim3(kPrepBlock), 0, st, a.theta,
                           a.vd, a.n_points, staged, a.o.bits, n_words, a.off, a.n_clusters,
                           best_key, hist);
        hipLaunchKernelGGL(batch_scatter_kernel,
                           dim3((unsigned)((a.n_clusters + kPrepBlock - 1) / kPrepBlock)),
                           dim3(kPrepBlock), 0, st, a.off, a.n_clusters, a.n_points, bt, tune,
                           (const uint32_t *)hist, queues, n_big, desc);
    }
    if (timed) (void)hipEventRecord(tc.ev[1], st);
    hipLaunchKernelGGL(batch_score(a.tuning.fp16_min_points > 0, plan.block), dim3(grid),
                       dim3(plan.block), 0, st, (const ItemDesc *)desc, a.n_clusters, a.n_hyp,
                       plan.rounds, plan.parts, plan.prune, plan.defer, pts, a.tau, queues, best_key,
                       a.o.hyp_counts);
    if (timed) (void)hipEventRecord(tc.ev[2], st);
    launch_refit(true, nullptr, nullptr, desc, a.n_clusters, n_big, a.n_points, a.n_hyp, 0, 0, 0, 0,
                 pts, best_key, a.tau, a.o, kNoneDone, plan.block == kLongBlock, plan.defer, st);
    if (timed) {
        (void)hipEventRecord(tc.ev[3], st);
        keep_timed_call(tc);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    return RV_OK;
}

BatchArgs make_batch_args(const float *theta, const float *vd, const int32_t *cluster_offsets,
                          const int32_t *frame_offsets, const uint64_t *seeds, int64_t n_frames,
                          int64_t n_clusters, int64_t n_points, int32_t n_hyp, float tau,
                          float *vx, float *vy, float *heading, int32_t *n_inliers,
                          uint8_t *status, int32_t *n_near_tau, uint32_t *inlier_bits,
                          int32_t *hyp_counts, int32_t *best_hyp, const rv_tuning_t *tuning,
                          void *workspace, size_t workspace_bytes) {
    BatchArgs a;
    a.theta = theta;
    a.vd = vd;
    a.off = cluster_offsets;
    a.frame_off = frame_offsets;
    a.seeds = seeds;
    a.n_frames = n_frames;
    a.n_clusters = n_clusters;
    a.n_points = n_points;
    a.n_hyp = n_hyp;
    a.tau = tau;
    a.o.vx = vx;
    a.o.vy = vy;
    a.o.heading = heading;
    a.o.n_inliers = n_inliers;
    a.o.status = status;
    a.o.n_near = n_near_tau;
    a.o.best = best_hyp;
    a.o.hyp_counts = hyp_counts;
    a.o.bits = inlier_bits;
    if (tuning != nullptr)
        a.tuning = *tuning;
    else
        rv_tuning_default(&a.tuning);
    a.workspace = workspace;
    a.workspace_bytes = workspace_bytes;
    return a;
}

// rv_estimate_velocity's checks and launches; allow_timing: record stage events
// when rv_stage_timing is on (the allocation-free entry point never does, since
// a first event set is created on demand).
int estimate_frame(const float *theta, const float *vd, const int32_t *cluster_offsets,
                   int64_t n_clusters, int64_t n_points, int32_t n_hyp, float tau, uint64_t seed,
                   float *vx, float *vy, float *heading, int32_t *n_inliers, uint8_t *status,
                   int32_t *n_near_tau, uint32_t *inlier_bits, int32_t *hyp_counts,
                   int32_t *best_hyp, void *workspace, size_t workspace_bytes, void *stream,
                   uint32_t first_cluster, int64_t first_point, bool allow_timing) {
    if (n_clusters < 0) return fail(RV_ERR_INVALID_ARG, "n_clusters < 0");
    if ((uint64_t)first_cluster + (uint64_t)n_clusters > ((uint64_t)1 << 32))
        return fail(RV_ERR_INVALID_ARG, "first_cluster + n_clusters exceeds 2^32");
    if (n_points < 0 || n_points > INT32_MAX)
        return fail(RV_ERR_INVALID_ARG, "n_points must be in [0, 2^31 - 1]");
    if (n_hyp < 1 || n_hyp > RV_MAX_HYP)
        return fail(RV_ERR_INVALID_ARG, "n_hyp must be in [1, %d]", RV_MAX_HYP);
    if (!(tau > 0.0f) || !isfinite(tau))
        return fail(RV_ERR_INVALID_ARG, "tau must be finite and > 0");
    if (cluster_offsets == nullptr) return fail(RV_ERR_INVALID_ARG, "cluster_offsets is NULL");
    if (n_points > 0 && (theta == nullptr || vd == nullptr))
        return fail(RV_ERR_INVALID_ARG, "theta or vd is NULL");
    if (n_clusters > 0 &&
        (vx == nullptr || vy == nullptr || heading == nullptr || n_inliers == nullptr ||
         status == nullptr))
        return fail(RV_ERR_INVALID_ARG, "a required output is NULL");
    const int64_t blocks_per_cluster = blocks_of(n_hyp);
    const int64_t clusters_xcd = (n_clusters + kXcds - 1) / kXcds * kXcds;
    if (clusters_xcd > (int64_t)INT32_MAX / blocks_per_cluster)
        return fail(RV_ERR_INVALID_ARG, "n_clusters * ceil(n_hyp / 256) exceeds 2^31 - 1");
    const Layout L = make_layout(n_clusters, n_points);
    if (workspace == nullptr || workspace_bytes < L.total)
        return fail(RV_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", L.total,
                    workspace == nullptr ? (size_t)0 : workspace_bytes);
    if (((uintptr_t)workspace % kAlign) != 0)
        return fail(RV_ERR_WORKSPACE, "workspace must be %zu-byte aligned", kAlign);
    if (n_clusters == 0) return RV_OK;

    char *ws = (char *)workspace;
    const Staging staged = {(StagedPoint *)(ws + L.staged), (StagedLow *)(ws + L.low)};
    Points pts;
    pts.staged = staged.points;
    pts.low = staged.low;
    pts.theta = theta;
    int32_t *order = n_clusters <= kPlanMaxClusters ? (int32_t *)(ws + L.order) : nullptr;
    int64_t *n_big = (int64_t *)(ws + L.n_big);
    unsigned long long *best_key = (unsigned long long *)(ws + L.best_key);
    const uint32_t key0 = (uint32_t)(seed & 0xFFFFFFFFu), key1 = (uint32_t)(seed >> 32);
    const int64_t n_words = inlier_bits != nullptr ? (n_points + 31) / 32 : 0;
    hipStream_t st = (hipStream_t)stream;

    Outputs o;
    o.vx = vx;
    o.vy = vy;
    o.heading = heading;
    o.n_inliers = n_inliers;
    o.status = status;
    o.n_near = n_near_tau;
    o.best = best_hyp;
    o.hyp_counts = hyp_counts;
    o.bits = inlier_bits;

    TimedCall tc;
    const bool timed = allow_timing && take_timed_call(tc);
    if (timed) (void)hipEventRecord(tc.ev[0], st);
    if (use_cluster_path(n_clusters, n_points, n_hyp, inlier_bits)) {
        // One launch; its time counts as the scoring stage.
        if (timed) (void)hipEventRecord(tc.ev[1], st);
        hipLaunchKernelGGL(cluster_kernel, dim3((unsigned)n_clusters), dim3(kScoreBlock), 0, st,
                           theta, vd, cluster_offsets, n_points, n_hyp, key0, key1, first_cluster,
                           first_point, small_to(1, tau, kSingleLanesMax), prune_from(1, tau, hyp_counts),
                           tau, staged, o);
        if (timed) {
            (void)hipEventRecord(tc.ev[2], st);
            (void)hipEventRecord(tc.ev[3], st);
            keep_timed_call(tc);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(RV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
        return RV_OK;
    }
    const ScorePlan plan =
        plan_score(n_clusters, n_points, n_hyp, tau, hyp_counts, kSingleLanesMax, 0);
    const bool many = n_clusters >= kRefitManyClusters;
    const bool refit_big = plan.parts == 1 && many && order != nullptr;  // the order counts them
    const bool split = refit_big && plan.rounds == kPruneHyp / kScoreBlock;
    const int32_t parts = split ? kSplitParts : plan.parts;
    int64_t score_blocks = clusters_xcd * parts;
    if (split) score_blocks = n_clusters + (parts - 1) * split_max(n_clusters, n_points);
    const bool defer = plan.defer && order != nullptr;
    int64_t prep_items = n_points > n_words ? n_points : n_words;
    prep_items = prep_items > n_clusters ? prep_items : n_clusters;
    const int64_t prep_blocks = (prep_items + kPrepBlock - 1) / kPrepBlock + 1;  // + planner
    hipLaunchKernelGGL(prep_kernel, dim3((unsigned)prep_blocks), dim3(kPrepBlock), 0, st, theta,
                       vd, n_points, staged, inlier_bits, n_words, cluster_offsets,
                       first_point, n_clusters, refit_big_class(n_clusters),
                       order, n_big, best_key);
    if (timed) (void)hipEventRecord(tc.ev[1], st);
    hipLaunchKernelGGL(plan.block == kLongBlock ? score_kernel<kLongBlock>
                                                : score_kernel<kScoreBlock>,
                       dim3((unsigned)score_blocks), dim3(plan.block), 0, st,
                       cluster_offsets, order, n_clusters, n_points, n_hyp,
                       split ? plan.rounds / parts : plan.rounds, parts, key0, key1, first_cluster,
                       first_point, plan.small_max, plan.prune, pts, tau, best_key, o, refit_big,
                       split ? (const int64_t *)n_big + 1 : nullptr, defer);
    if (timed) (void)hipEventRecord(tc.ev[2], st);
    launch_refit(false, cluster_offsets, order, nullptr, n_clusters,
                 order != nullptr ? (const int64_t *)n_big : nullptr, n_points, n_hyp, key0, key1,
                 first_cluster, first_point, pts, best_key, tau, o, 
                 !refit_big ? kNoneDone : split ? kUnsplitDone : kBigDone, plan.block == kLongBlock, defer, st);
    if (timed) {
        (void)hipEventRecord(tc.ev[3], st);
        keep_timed_call(tc);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    return RV_OK;
}

// ---- Allocation-free single-frame entry point ------------------------------
//
// rv_estimate_velocity_noalloc keeps its workspace in `scratch`, a device array
// of RV_NOALLOC_SCRATCH_BYTES that each GPU holds from the load of this code
// object on it until the process ends.  In host code the array's name denotes a host-side
// stand-in, not device memory: host code only passes on the address that
// hipGetSymbolAddress returns for the current device, looked up once per device
// and kept in g_scratch.  Every kernel writes the parts of the workspace it
// reads before reading them (staged points, dispatch order, best keys), so the
// contents a previous call left need no clearing.
static __device__ __align__(256) unsigned char scratch[RV_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch[kMaxDevices];

// Device address of `scratch` on the device of `stream` (which must be the
// current device: the symbol is looked up with that device current).
int device_scratch(hipStream_t stream, void **ptr) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(RV_ERR_HIP, "hipGetDevice failed: %s", hipGetErrorString(e));
    if (stream != nullptr) {
        int sdev = -1;
        e = hipStreamGetDevice(stream, &sdev);
        if (e != hipSuccess)
            return fail(RV_ERR_HIP, "hipStreamGetDevice failed: %s", hipGetErrorString(e));
        if (sdev != dev)
            return fail(RV_ERR_INVALID_ARG,
                        "stream belongs to device %d, the current device is %d", sdev, dev);
    }
    if (dev < 0 || dev >= kMaxDevices)
        return fail(RV_ERR_HIP, "device index %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch[dev] == nullptr) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr)
            return fail(RV_ERR_HIP, "hipGetSymbolAddress(scratch) failed: %s",
                        hipGetErrorString(e));
        g_scratch[dev] = p;
    }
    *ptr = g_scratch[dev];
    return RV_OK;
}

// ---- A frame sent and estimated in parts ---------------------------------------
// Events that order a part's estimate after its copy, kept per device and
// reused: a wait enqueued on a stream holds on to the record that precedes it,
// so an event may go back to the pool as soon as its wait is enqueued.
std::mutex g_event_mutex;
std::vector<hipEvent_t> g_events[kMaxDevices];

int take_events(int dev, int n, hipEvent_t *ev) {
    std::lock_guard<std::mutex> lock(g_event_mutex);
    std::vector<hipEvent_t> &pool = g_events[dev];
    for (int i = 0; i < n; ++i) {
        if (pool.empty()) {
            const hipError_t e = hipEventCreateWithFlags(&ev[i], hipEventDisableTiming);
            if (e != hipSuccess) {
                for (int j = 0; j < i; ++j) pool.push_back(ev[j]);
                return fail(RV_ERR_HIP, "hipEventCreateWithFlags failed: %s",
                            hipGetErrorString(e));
            }
        } else {
            ev[i] = pool.back();
            pool.pop_back();
        }
    }
    return RV_OK;
}

void give_events(int dev, int n, const hipEvent_t *ev) {
    std::lock_guard<std::mutex> lock(g_event_mutex);
    for (int i = 0; i < n; ++i) g_events[dev].push_back(ev[i]);
}

// Clusters [cut[j], cut[j+1]) form part j.  Part j gets a share of the points
// proportional to n_parts - j (shares P, P - 1, ..., 1 out of P (P + 1) / 2):
// only the last part's estimate is not hidden behind a later copy, so the
// parts shrink toward the end.  The first cluster that starts at or after part
// j's first point starts it (parts without clusters are dropped).  Returns the
// number of parts.
int cut_parts(const int32_t *off, int64_t n_clusters, int64_t n_points, int n_parts,
              int64_t *cut) {
    int m = 0;
    cut[m++] = 0;
    int64_t k = 0;
    const int64_t total = (int64_t)n_parts * (n_parts + 1);
    for (int j = 1; j < n_parts; ++j) {
        const int64_t target = n_points * ((int64_t)j * (2 * n_parts - j + 1)) / total;
        while (k < n_clusters && off[k] < target) ++k;
        if (k > cut[m - 1] && k < n_clusters) cut[m++] = k;
    }
    cut[m++] = n_clusters;  // n_clusters > 0: every cut above is below it
    return m - 1;
}

int estimate_pipelined(const float *theta_host, const float *vd_host,
                       const int32_t *offsets_host, int64_t n_clusters, int64_t n_points,
                       int32_t n_parts, int32_t n_hyp, float tau, uint64_t seed, float *theta_dev,
                       float *vd_dev, int32_t *offsets_dev, float *vx, float *vy, float *heading,
                       int32_t *n_inliers, uint8_t *status, int32_t *n_near_tau,
                       int32_t *hyp_counts, int32_t *best_hyp, void *workspace,
                       size_t workspace_bytes, hipStream_t st, hipStream_t copy_st) {
    if (n_clusters < 0 || n_points < 0 || n_points > INT32_MAX)
        return fail(RV_ERR_INVALID_ARG, "sizes out of range");
    if (n_parts < 1 || n_parts > RV_MAX_PARTS)
        return fail(RV_ERR_INVALID_ARG, "n_parts must be in [1, %d]", RV_MAX_PARTS);
    if (offsets_host == nullptr || offsets_dev == nullptr)
        return fail(RV_ERR_INVALID_ARG, "offsets pointers are NULL");
    if (n_points > 0 && (theta_host == nullptr || vd_host == nullptr || theta_dev == nullptr ||
                         vd_dev == nullptr))
        return fail(RV_ERR_INVALID_ARG, "theta or vd pointers are NULL");
    // The host reads the offsets to cut the frame and to size the copies, so
    // they must describe the frame exactly.
    if (offsets_host[0] != 0 || offsets_host[n_clusters] != n_points)
        return fail(RV_ERR_INVALID_ARG, "offsets must start at 0 and end at n_points");
    for (int64_t k = 0; k < n_clusters; ++k)
        if (offsets_host[k + 1] < offsets_host[k])
            return fail(RV_ERR_INVALID_ARG, "offsets decrease at cluster %lld", (long long)k);
    if (n_clusters == 0) return RV_OK;
    if (workspace_bytes < rv_workspace_bytes(n_clusters, n_points, n_hyp))
        return fail(RV_ERR_WORKSPACE, "workspace of %zu bytes, %zu needed", workspace_bytes,
                    rv_workspace_bytes(n_clusters, n_points, n_hyp));
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(RV_ERR_HIP, "hipGetDevice failed: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(RV_ERR_HIP, "device index %d outside [0, %d)", dev, kMaxDevices);
    int64_t cut[RV_MAX_PARTS + 1];
    const int m = cut_parts(offsets_host, n_clusters, n_points, n_parts, cut);
    hipEvent_t ev[RV_MAX_PARTS + 1];
    int rc = take_events(dev, m + 1, ev);
    if (rc != RV_OK) return rc;
    // The copies wait for the work already queued on `stream` (a previous
    // call's estimates may still read the same device buffers); then every
    // copy is enqueued first, so that the copy engine never waits for the
    // host, and each part's estimate behind its copy.
    e = hipEventRecord(ev[m], st);
    if (e == hipSuccess) e = hipStreamWaitEvent(copy_st, ev[m], 0);
    if (e == hipSuccess)
        e = hipMemcpyAsync(offsets_dev, offsets_host, (size_t)(n_clusters + 1) * sizeof(int32_t),
                           hipMemcpyHostToDevice, copy_st);
    for (int j = 0; j < m && e == hipSuccess; ++j) {
        const int64_t p0 = offsets_host[cut[j]], p1 = offsets_host[cut[j + 1]];
        if (p1 > p0) {
            e = hipMemcpyAsync(theta_dev + p0, theta_host + p0, (size_t)(p1 - p0) * sizeof(float),
                               hipMemcpyHostToDevice, copy_st);
            if (e == hipSuccess)
                e = hipMemcpyAsync(vd_dev + p0, vd_host + p0, (size_t)(p1 - p0) * sizeof(float),
                                   hipMemcpyHostToDevice, copy_st);
        }
        if (e == hipSuccess) e = hipEventRecord(ev[j], copy_st);
    }
    for (int j = 0; j < m && e == hipSuccess && rc == RV_OK; ++j) {
        e = hipStreamWaitEvent(st, ev[j], 0);
        if (e != hipSuccess) break;
        const int64_t c0 = cut[j], c1 = cut[j + 1];
        const int64_t p0 = offsets_host[c0], p1 = offsets_host[c1];
        rc = estimate_frame(theta_dev + p0, vd_dev + p0, offsets_dev + c0, c1 - c0, p1 - p0, n_hyp,
                            tau, seed, vx + c0, vy + c0, heading + c0, n_inliers + c0,
                            status + c0, n_near_tau != nullptr ? n_near_tau + c0 : nullptr,
                            nullptr, hyp_counts != nullptr ? hyp_counts + c0 * n_hyp : nullptr,
                            best_hyp != nullptr ? best_hyp + c0 : nullptr, workspace,
                            workspace_bytes, (void *)st, (uint32_t)c0, p0, false);
    }
    give_events(dev, m + 1, ev);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(RV_ERR_HIP, "pipelined copy or wait failed: %s", hipGetErrorString(e));
    }
    return rc;
}

}  // namespace

extern "C" {

size_t rv_workspace_bytes(int64_t n_clusters, int64_t n_points, int32_t n_hyp) {
    if (n_clusters < 0 || n_points < 0 || n_hyp < 0) return 0;
    return make_layout(n_clusters, n_points).total;
}

const char *rv_last_error(void) { return g_error; }

int rv_estimate_velocity(const float *theta, const float *vd, const int32_t *cluster_offsets,
                         int64_t n_clusters, int64_t n_points, int32_t n_hyp, float tau,
                         uint64_t seed, float *vx, float *vy, float *heading, int32_t *n_inliers,
                         uint8_t *status, int32_t *n_near_tau, uint32_t *inlier_bits,
                         int32_t *hyp_counts, int32_t *best_hyp, void *workspace,
                         size_t workspace_bytes, void *stream) {
    g_error[0] = '\0';
    return estimate_frame(theta, vd, cluster_offsets, n_clusters, n_points, n_hyp, tau, seed, vx,
                          vy, heading, n_inliers, status, n_near_tau, inlier_bits, hyp_counts,
                          best_hyp, workspace, workspace_bytes, stream, 0u, 0, true);
}

int rv_estimate_velocity_part(const float *theta, const float *vd, const int32_t *cluster_offsets,
                              int64_t n_clusters, int64_t n_points, int64_t first_cluster,
                              int64_t first_point, int32_t n_hyp, float tau, uint64_t seed,
                              float *vx, float *vy, float *heading, int32_t *n_inliers,
                              uint8_t *status, int32_t *n_near_tau, uint32_t *inlier_bits,
                              int32_t *hyp_counts, int32_t *best_hyp, void *workspace,
                              size_t workspace_bytes, void *stream) {
    g_error[0] = '\0';
    if (first_cluster < 0 || first_cluster > (int64_t)UINT32_MAX)
        return fail(RV_ERR_INVALID_ARG, "first_cluster must be in [0, 2^32 - 1]");
    if (first_point < 0 || first_point > INT32_MAX)
        return fail(RV_ERR_INVALID_ARG, "first_point must be in [0, 2^31 - 1]");
    return estimate_frame(theta, vd, cluster_offsets, n_clusters, n_points, n_hyp, tau, seed, vx,
                          vy, heading, n_inliers, status, n_near_tau, inlier_bits, hyp_counts,
                          best_hyp, workspace, workspace_bytes, stream, (uint32_t)first_cluster,
                          first_point, true);
}

int rv_estimate_velocity_pipelined(const float *theta_host, const float *vd_host,
                                   const int32_t *offsets_host, int64_t n_clusters,
                                   int64_t n_points, int32_t n_parts, int32_t n_hyp, float tau,
                                   uint64_t seed, float *theta_dev, float *vd_dev,
                                   int32_t *offsets_dev, float *vx, float *vy, float *heading,
                                   int32_t *n_inliers, uint8_t *status, int32_t *n_near_tau,
                                   int32_t *hyp_counts, int32_t *best_hyp, void *workspace,
                                   size_t workspace_bytes, void *stream, void *copy_stream) {
    g_error[0] = '\0';
    return estimate_pipelined(theta_host, vd_host, offsets_host, n_clusters, n_points, n_parts,
                              n_hyp, tau, seed, theta_dev, vd_dev, offsets_dev, vx, vy, heading,
                              n_inliers, status, n_near_tau, hyp_counts, best_hyp, workspace,
                              workspace_bytes, (hipStream_t)stream, (hipStream_t)copy_stream);
}

int rv_estimate_velocity_noalloc(const float *theta, const float *vd,
                                 const int32_t *cluster_offsets, int64_t n_clusters,
                                 int64_t n_points, int32_t n_hyp, float tau, uint64_t seed,
                                 float *vx, float *vy, float *heading, int32_t *n_inliers,
                                 uint8_t *status, int32_t *n_near_tau, uint32_t *inlier_bits,
                                 int32_t *hyp_counts, int32_t *best_hyp, void *stream) {
    g_error[0] = '\0';
    const size_t need = rv_workspace_bytes(n_clusters, n_points, n_hyp);
    if (need > RV_NOALLOC_SCRATCH_BYTES)
        return fail(RV_ERR_WORKSPACE,
                    "frame of %lld clusters and %lld points needs %zu bytes of workspace; the "
                    "allocation-free entry point holds %zu",
                    (long long)n_clusters, (long long)n_points, need,
                    (size_t)RV_NOALLOC_SCRATCH_BYTES);
    void *ws = nullptr;
    if (int rc = device_scratch((hipStream_t)stream, &ws)) return rc;
    return estimate_frame(theta, vd, cluster_offsets, n_clusters, n_points, n_hyp, tau, seed, vx,
                          vy, heading, n_inliers, status, n_near_tau, inlier_bits, hyp_counts,
                          best_hyp, ws, RV_NOALLOC_SCRATCH_BYTES, stream, 0u, 0, false);
}

int rv_stage_timing(int enable) {
    std::lock_guard<std::mutex> lock(g_timing_mutex);
    g_timing = enable != 0;
    return RV_OK;
}

int rv_stage_times(double *ms, int64_t *n_calls) {
    std::vector<TimedCall> calls;
    {
        std::lock_guard<std::mutex> lock(g_timing_mutex);
        calls.swap(g_pending);
    }
    double sum[kStages] = {0.0, 0.0, 0.0};
    int rc = RV_OK;
    for (const TimedCall &tc : calls) {
        if (hipEventSynchronize(tc.ev[kStages]) != hipSuccess) {
            rc = fail(RV_ERR_HIP, "hipEventSynchronize failed");
            continue;
        }
        for (int s = 0; s < kStages; ++s) {
            float t = 0.0f;
            if (hipEventElapsedTime(&t, tc.ev[s], tc.ev[s + 1]) != hipSuccess) {
                rc = fail(RV_ERR_HIP, "hipEventElapsedTime failed");
                continue;
            }
            sum[s] += t;
        }
    }
    {
        std::lock_guard<std::mutex> lock(g_timing_mutex);
        g_free.insert(g_free.end(), calls.begin(), calls.end());
    }
    if (ms)
        for (int s = 0; s < kStages; ++s) ms[s] = sum[s];
    if (n_calls) *n_calls = (int64_t)calls.size();
    return rc;
}

int rv_host_device_pointer(const void *host_ptr, void **device_ptr) {
    g_error[0] = '\0';
    if (device_ptr == nullptr) return fail(RV_ERR_INVALID_ARG, "device_ptr is NULL");
    *device_ptr = nullptr;
    if (host_ptr == nullptr) return fail(RV_ERR_INVALID_ARG, "host_ptr is NULL");
    hipPointerAttribute_t attr;
    hipError_t e = hipPointerGetAttributes(&attr, host_ptr);
    if (e != hipSuccess || attr.type != hipMemoryTypeHost) {
        (void)hipGetLastError();  // a failed query leaves its error behind
        return fail(RV_ERR_INVALID_ARG, "%p is not pinned host memory (hipHostMalloc)", host_ptr);
    }
    void *d = nullptr;
    e = hipHostGetDevicePointer(&d, const_cast<void *>(host_ptr), 0);
    if (e != hipSuccess || d == nullptr) {
        (void)hipGetLastError();
        return fail(RV_ERR_INVALID_ARG, "no device mapping of %p: %s", host_ptr,
                    hipGetErrorString(e));
    }
    *device_ptr = d;
    return RV_OK;
}

int rv_philox4x32_10(const uint32_t *ctr, const uint32_t *key, uint32_t *out, int64_t n,
                     void *stream) {
    g_error[0] = '\0';
    if (n < 0) return fail(RV_ERR_INVALID_ARG, "n < 0");
    if (n == 0) return RV_OK;
    if (ctr == nullptr || key == nullptr || out == nullptr)
        return fail(RV_ERR_INVALID_ARG, "a pointer is NULL");
    const int64_t grid = (n + kPrepBlock - 1) / kPrepBlock;
    if (grid > INT32_MAX) return fail(RV_ERR_INVALID_ARG, "n too large");
    hipLaunchKernelGGL(philox_kernel, dim3((unsigned)grid), dim3(kPrepBlock), 0,
                       (hipStream_t)stream, ctr, key, out, n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    return RV_OK;
}


void rv_tuning_default(rv_tuning_t *t) {
    if (t == nullptr) return;
    for (int b = 0; b < RV_TUNE_BUCKETS; ++b) t->rows_max[b] = kRowsMax;
    t->blocks_per_cu = 0;
    t->fp16_min_points = 0;
    t->lanes_max_points = kDefaultLanesMax;
}

size_t rv_batch_workspace_bytes(int64_t n_frames, int64_t n_clusters, int64_t n_points,
                                int32_t n_hyp) {
    if (n_frames < 1 || n_clusters < 0 || n_points < 0 || n_hyp < 0) return 0;
    return make_batch_layout(n_clusters, n_points).total;
}

int rv_estimate_velocity_batch(const float *theta, const float *vd, const int32_t *cluster_offsets,
                               const int32_t *frame_offsets, const uint64_t *seeds,
                               int64_t n_frames, int64_t n_clusters, int64_t n_points,
                               int32_t n_hyp, float tau, float *vx, float *vy, float *heading,
                               int32_t *n_inliers, uint8_t *status, int32_t *n_near_tau,
                               uint32_t *inlier_bits, int32_t *hyp_counts, int32_t *best_hyp,
                               const rv_tuning_t *tuning, void *workspace,
                               size_t workspace_bytes, void *stream) {
    g_error[0] = '\0';
    const BatchArgs a = make_batch_args(theta, vd, cluster_offsets, frame_offsets, seeds,
                                        n_frames, n_clusters, n_points, n_hyp, tau, vx, vy,
                                        heading, n_inliers, status, n_near_tau, inlier_bits,
                                        hyp_counts, best_hyp, tuning, workspace, workspace_bytes);
    if (int rc = check_batch(a)) return rc;
    unsigned grid = 1;
    if (int rc = persistent_blocks(a, &grid)) return rc;
    return launch_batch(a, grid, (hipStream_t)stream, true);
}

struct rv_graph {
    hipGraph_t graph;
    hipGraphExec_t exec;
};

int rv_graph_capture_batch(const float *theta, const float *vd, const int32_t *cluster_offsets,
                           const int32_t *frame_offsets, const uint64_t *seeds, int64_t n_frames,
                           int64_t n_clusters, int64_t n_points, int32_t n_hyp, float tau,
                           float *vx, float *vy, float *heading, int32_t *n_inliers,
                           uint8_t *status, int32_t *n_near_tau, uint32_t *inlier_bits,
                           int32_t *hyp_counts, int32_t *best_hyp, const rv_tuning_t *tuning,
                           void *workspace, size_t workspace_bytes, rv_graph_t **graph) {
    g_error[0] = '\0';
    if (graph == nullptr) return fail(RV_ERR_INVALID_ARG, "graph is NULL");
    *graph = nullptr;
    const BatchArgs a = make_batch_args(theta, vd, cluster_offsets, frame_offsets, seeds,
                                        n_frames, n_clusters, n_points, n_hyp, tau, vx, vy,
                                        heading, n_inliers, status, n_near_tau, inlier_bits,
                                        hyp_counts, best_hyp, tuning, workspace, workspace_bytes);
    if (int rc = check_batch(a)) return rc;
    unsigned grid = 1;
    if (int rc = persistent_blocks(a, &grid)) return rc;
    hipStream_t cap = nullptr;
    if (hipStreamCreateWithFlags(&cap, hipStreamNonBlocking) != hipSuccess)
        return fail(RV_ERR_HIP, "hipStreamCreate failed");
    rv_graph_t *g = new rv_graph_t;
    g->graph = nullptr;
    g->exec = nullptr;
    int rc = RV_OK;
    if (hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
        rc = fail(RV_ERR_HIP, "hipStreamBeginCapture failed");
    } else {
        rc = launch_batch(a, grid, cap, false);
        const hipError_t e = hipStreamEndCapture(cap, &g->graph);
        if (rc == RV_OK && e != hipSuccess)
            rc = fail(RV_ERR_HIP, "hipStreamEndCapture failed: %s", hipGetErrorString(e));
        if (rc == RV_OK && hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0) != hipSuccess)
            rc = fail(RV_ERR_HIP, "hipGraphInstantiate failed");
    }
    (void)hipStreamDestroy(cap);
    if (rc != RV_OK) {
        rv_graph_destroy(g);
        return rc;
    }
    *graph = g;
    return RV_OK;
}

int rv_graph_launch(rv_graph_t *graph, void *stream) {
    g_error[0] = '\0';
    if (graph == nullptr || graph->exec == nullptr) return fail(RV_ERR_INVALID_ARG, "graph is NULL");
    const hipError_t e = hipGraphLaunch(graph->exec, (hipStream_t)stream);
    if (e != hipSuccess) return fail(RV_ERR_HIP, "hipGraphLaunch failed: %s", hipGetErrorString(e));
    return RV_OK;
}

void rv_graph_destroy(rv_graph_t *graph) {
    if (graph == nullptr) return;
    if (graph->exec != nullptr) (void)hipGraphExecDestroy(graph->exec);
    if (graph->graph != nullptr) (void)hipGraphDestroy(graph->graph);
    delete graph;
}

}  // extern "C"
