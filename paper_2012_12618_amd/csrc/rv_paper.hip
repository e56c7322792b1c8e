// rv_paper.hip -- gfx950 kernels and host entry point of the paper-literal
// variant of the inlier kernel (Sec. 3.1, Alg. 1 with Eq. 5's threshold),
// followed by the least-squares kernel (Sec. 3.2, Eq. 7, Alg. 2, Eq. 8).
//
// Per cluster:
//   stats   one workgroup: per-cluster min-max normalisation of azimuth and
//           Doppler onto [0, 1] (Alg. 1's normalize(); a zero span maps to 0),
//           then the median absolute deviation of the normalised Doppler
//           values (Eq. 5, read as the statistic the text names): two medians,
//           each selected from a histogram in LDS; clears its share of the
//           frame-wide inlier mask.
//   score   a thread per (trial, cluster) draws the trial's seed pair from
//           Philox4x32-10 exactly as the velocity-profile kernels do and fits the
//           line through the two normalised seeds (Alg. 1); then the workgroup's
//           waves share the cluster's points, every lane counting those whose
//           perpendicular distance (aa x + bb y + cc over sqrt(aa^2 + bb^2)) is at
//           most the threshold (for each line, as one comparison of the numerator
//           against the largest value that passes, found once per trial); the
//           block's best (count, lowest index) key is merged per cluster with a
//           64-bit atomic maximum.
//   refit   one workgroup: re-classifies every point under the kept line,
//           writes the inlier mask, and solves the normal equations of the
//           velocity profile on the inliers; heading = atan2(vy, vx).
// Each step is a device function.  Calls that ask for the frame-wide inlier
// mask, or have more than 256 trials per cluster, or frames above 65,536
// points or clusters, run them as three kernels; all others run them in one
// kernel, a workgroup per cluster, with the same results bit for bit.
//
// Everything is FP64 and evaluated exactly as written (no contraction), so
// counts, masks and thresholds are the same bits as a plain FP64 evaluation of
// the same expressions.

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include "rv.h"
#include "rv_device.h"
#include "rv_internal.h"

#pragma clang fp contract(off)

using rv_internal::fail;
using rv_internal::g_error;
using rv_internal::keep_timed_call;
using rv_internal::take_timed_call;
using rv_internal::TimedCall;

namespace {

constexpr int kPaperBlock = 256;
constexpr int kPaperWaves = kPaperBlock / kWave;
constexpr double kPaperMinSeparation = RV_MIN_SEED_SEPARATION;

// Normalised coordinate of one value: (a - lo) / span, 0 for a zero span.
__device__ __forceinline__ double unit_coord(float a, double lo, double span) {
    return span > 0.0 ? ((double)a - lo) / span : 0.0;
}

// Spans of a cluster with 2 <= n <= RV_PAPER_MAX_POINTS points, the only ones
// the score and refit kernels work on.
__device__ __forceinline__ bool paper_cluster(const Span &sp) {
    return sp.ok && sp.n >= 2 && sp.n <= RV_PAPER_MAX_POINTS;
}

constexpr int kSelectBins = 1024;
constexpr int64_t kClearWords = 2048;  // words of the mask per clearing workgroup, at most

// Workgroup LDS of the threshold step.
struct StatsShared {
    uint32_t hist[kSelectBins];
    double sel[kPaperBlock];
    float red[4][kPaperWaves];
    uint32_t cnt[kPaperWaves];
    uint32_t bin[2], below, n_sel;
    double mid[2];
};

// Bins of the histogram that hold the positions q0 <= q1 in sorted order, into
// sh.bin, and the number of entries below the first, into sh.below.  Called by the
// whole workgroup after a barrier; ends with one.
__device__ __forceinline__ void find_bins(StatsShared &sh, uint32_t q0, uint32_t q1) {
    constexpr int kEach = kSelectBins / kPaperBlock;
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kEach; ++i) sum += sh.hist[tid * kEach + i];
    const uint32_t incl = wave_inclusive_sum(sum);
    if (lane == kWave - 1) sh.cnt[wave] = incl;
    __syncthreads();
    uint32_t at = incl - sum;
    for (int w = 0; w < wave; ++w) at += sh.cnt[w];
#pragma unroll
    for (int i = 0; i < kEach; ++i) {
        const uint32_t end = at + sh.hist[tid * kEach + i];
        if (at <= q0 && q0 < end) {
            sh.bin[0] = tid * kEach + i;
            sh.below = at;
        }
        if (at <= q1 && q1 < end) sh.bin[1] = tid * kEach + i;
        at = end;
    }
    __syncthreads();
}

// Median (mean of the two middle values for an even count) of the m values
// value(p) in [0, 1] over the points p < n for which it is not NaN, m >= 1, without
// sorting: a histogram of the values (monotone bins) finds the bins that hold the
// middle positions; their entries, usually a handful, are ranked against each
// other, and the entry whose rank range holds a middle position is that order
// statistic (equal entries write the same value).  When more than kPaperBlock
// entries share those bins (many equal values), the two order statistics are
// selected digit by digit of their bit patterns instead (non-negative doubles order
// like them).  A bitonic sort of 2048 values took 66 barriers; this takes six.
// Whole workgroup.
template <typename Value>
__device__ __forceinline__ double select_median(StatsShared &sh, int n, int m, const Value &value) {
    const int tid = threadIdx.x;
    const uint32_t q1 = m / 2, q0 = (m & 1) ? q1 : q1 - 1;
    const auto bin_of = [](double y) {
        const int b = (int)(y * kSelectBins);
        return (uint32_t)(b < kSelectBins - 1 ? b : kSelectBins - 1);
    };
    for (int i = tid; i < kSelectBins; i += kPaperBlock) sh.hist[i] = 0;
    if (tid == 0) sh.n_sel = 0;
    __syncthreads();
    for (int p = tid; p < n; p += kPaperBlock) {
        const double y = value(p);
        if (!__builtin_isnan(y)) atomicAdd(&sh.hist[bin_of(y)], 1u);
    }
    __syncthreads();
    find_bins(sh, q0, q1);
    const uint32_t b0 = sh.bin[0], b1 = sh.bin[1], below = sh.below;
    for (int p = tid; p < n; p += kPaperBlock) {
        const double y = value(p);
        if (!__builtin_isnan(y) && bin_of(y) >= b0 && bin_of(y) <= b1) {
            const uint32_t k = atomicAdd(&sh.n_sel, 1u);
            if (k < kPaperBlock) sh.sel[k] = y;
        }
    }
    __syncthreads();
    const uint32_t n_sel = sh.n_sel;
    if (n_sel <= kPaperBlock) {
        if ((uint32_t)tid < n_sel) {
            const double a = sh.sel[tid];
            uint32_t lo = below, hi = below;
            for (uint32_t j = 0; j < n_sel; ++j) {
                const double b = sh.sel[j];
                lo += b < a ? 1u : 0u;
                hi += b <= a ? 1u : 0u;
            }
            if (lo <= q0 && q0 < hi) sh.mid[0] = a;
            if (lo <= q1 && q1 < hi) sh.mid[1] = a;
        }
        __syncthreads();
    } else {
        for (int which = 0; which < 2; ++which) {
            uint32_t k = which == 0 ? q0 : q1;
            uint64_t prefix = 0;
            for (int bits = 64; bits > 0;) {
                const int width = bits < 10 ? bits : 10;
                bits -= width;
                __syncthreads();
                for (int i = tid; i < kSelectBins; i += kPaperBlock) sh.hist[i] = 0;
                __syncthreads();
                for (int p = tid; p < n; p += kPaperBlock) {
                    const double y = value(p);
                    const uint64_t u = __builtin_bit_cast(uint64_t, y);
                    if (!__builtin_isnan(y) && (bits + width == 64 || (u >> (bits + width)) == prefix))
                        atomicAdd(&sh.hist[(u >> bits) & ((1u << width) - 1u)], 1u);
                }
                __syncthreads();
                find_bins(sh, k, k);
                prefix = (prefix << width) | sh.bin[0];
                k -= sh.below;
            }
            if (tid == 0) sh.mid[which] = __builtin_bit_cast(double, prefix);
        }
        __syncthreads();
    }
    const double lo = sh.mid[0], hi = sh.mid[1];
    __syncthreads();
    return (m & 1) ? hi : (lo + hi) / 2.0;
}

// Threshold step of cluster k (whole workgroup; uniform early returns): the
// normalised (x, y) of its points into xy (and into s_xy, when given, for
// clusters of at most kPaperBlock points), and its threshold into thresh[k],
// NaN when the cluster takes no part or has no usable point.  Returns the
// threshold in every thread.
__device__ __forceinline__ double paper_stats(const float *__restrict__ theta, const float *__restrict__ vd,
                              Span sp, int64_t k, double2 *__restrict__ xy,
                              double *__restrict__ thresh, StatsShared &sh, double2 *s_xy) {
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    if (tid == 0) thresh[k] = __builtin_nan("");
    if (!paper_cluster(sp)) return __builtin_nan("");
    const int n = (int)sp.n;
    const float *t = theta + sp.lo, *v = vd + sp.lo;
    // Extremes of the finite points (the same in float32 as in FP64).
    float tmin = __builtin_inff(), tmax = -__builtin_inff();
    float vmin = __builtin_inff(), vmax = -__builtin_inff();
    uint32_t m_ok = 0;
    for (int p = tid; p < n; p += kPaperBlock) {
        const float tp = t[p], vp = v[p];
        if (!(isfinite(tp) && isfinite(vp))) continue;
        tmin = fminf(tmin, tp);
        tmax = fmaxf(tmax, tp);
        vmin = fminf(vmin, vp);
        vmax = fmaxf(vmax, vp);
        m_ok += 1;
    }
    tmin = wave_min_f(tmin);
    tmax = wave_max_f(tmax);
    vmin = wave_min_f(vmin);
    vmax = wave_max_f(vmax);
    m_ok = __builtin_amdgcn_readlane(wave_inclusive_sum(m_ok), kWave - 1);
    if (lane == 0) {
        sh.red[0][wave] = tmin;
        sh.red[1][wave] = tmax;
        sh.red[2][wave] = vmin;
        sh.red[3][wave] = vmax;
        sh.cnt[wave] = m_ok;
    }
    __syncthreads();
    tmin = sh.red[0][0];
    tmax = sh.red[1][0];
    vmin = sh.red[2][0];
    vmax = sh.red[3][0];
    m_ok = sh.cnt[0];
    for (int w = 1; w < kPaperWaves; ++w) {
        tmin = fminf(tmin, sh.red[0][w]);
        tmax = fmaxf(tmax, sh.red[1][w]);
        vmin = fminf(vmin, sh.red[2][w]);
        vmax = fmaxf(vmax, sh.red[3][w]);
        m_ok += sh.cnt[w];
    }
    const double tlo = tmin, tspan = (double)tmax - (double)tmin;
    const double vlo = vmin, vspan = (double)vmax - (double)vmin;

    // Normalised coordinates; NaN marks a point that takes no part.
    for (int p = tid; p < n; p += kPaperBlock) {
        const float tp = t[p], vp = v[p];
        const bool ok = isfinite(tp) && isfinite(vp);
        const double2 q = make_double2(ok ? unit_coord(tp, tlo, tspan) : __builtin_nan(""),
                                       ok ? unit_coord(vp, vlo, vspan) : __builtin_nan(""));
        xy[sp.lo + p] = q;
        if (s_xy != nullptr && n <= kPaperBlock) s_xy[p] = q;
    }
    if (m_ok == 0) return __builtin_nan("");
    // The thread's own values (it wrote them itself).
    const bool in_lds = s_xy != nullptr && n <= kPaperBlock;
    const auto y_of = [&](int p) { return in_lds ? s_xy[p].y : xy[sp.lo + p].y; };
    // The median of y (|y - 0|: no y is negative), then of |y - median|.
    double mid = 0.0;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        const double center = mid;
        mid = select_median(sh, n, (int)m_ok, [&](int p) { return fabs(y_of(p) - center); });
    }
    if (tid == 0) thresh[k] = mid;
    return mid;
}

__global__ __launch_bounds__(kPaperBlock) void paper_stats_kernel(
    const float *__restrict__ theta, const float *__restrict__ vd,
    const int32_t *__restrict__ off, int64_t n_clusters, int64_t n_points,
    double2 *__restrict__ xy, double *__restrict__ thresh,
    unsigned long long *__restrict__ best_key, uint32_t *__restrict__ bits, int64_t n_words) {
    __shared__ StatsShared sh;
    const int64_t k = blockIdx.x;
    // This workgroup's share of the frame-wide mask, cleared for the refit kernel.
    if (bits != nullptr) {
        const int64_t w1 = n_words * (k + 1) / gridDim.x;
        for (int64_t w = n_words * k / gridDim.x + threadIdx.x; w < w1; w += kPaperBlock) bits[w] = 0u;
    }
    if (k >= n_clusters) return;
    if (threadIdx.x == 0) best_key[k] = 0;
    (void)paper_stats(theta, vd, cluster_span(off, k, n_points), k, xy, thresh, sh, nullptr);
}

// Line of a trial through its normalised seeds (Alg. 1: slope and intercept)
// and the denominator of its distance.
struct Line {
    double m, c, distd;
    bool valid;
};

__device__ __forceinline__ Line trial_line(const float *__restrict__ t, const double2 *__restrict__ xy,
                                           int n, uint32_t h, uint32_t k, uint32_t key0,
                                           uint32_t key1) {
    const uint4 u = philox4x32_10(make_uint4(h, k, 0u, 0u), key0, key1);
    uint32_t i, j;
    seed_pair(u.x, u.y, (uint32_t)n, i, j);
    const double2 a = xy[i], b = xy[j];
    Line L;
    L.valid = !__builtin_isnan(a.x) && !__builtin_isnan(b.x) &&
              fabs((double)t[j] - (double)t[i]) >= kPaperMinSeparation;
    L.m = L.c = L.distd = 0.0;
    if (!L.valid) return L;
    L.m = (b.y - a.y) / (b.x - a.x);
    L.c = a.y - L.m * a.x;
    const double aa = -L.m, bb = 1.0;
    L.distd = sqrt(aa * aa + bb * bb);
    return L;
}

// Numerator of Alg. 1's distance, aa x + bb y + cc with aa = -m, bb = 1 and
// cc = -c, evaluated as written.
__device__ __forceinline__ double dist_num(const Line &L, double2 p) {
    const double aa = -L.m, bb = 1.0, cc = -L.c;
    return (aa * p.x + bb * p.y) + cc;
}

// Alg. 1's inlier test of one point against a valid line.
__device__ __forceinline__ bool within(const Line &L, double2 p, double th) {
    return fabs(dist_num(L, p) / L.distd) <= th;
}

// The same test without a division per point.  For one line, the rounded
// quotient |num| / distd is at most th exactly when |num| <= bound, the
// largest double x >= 0 whose quotient x / distd rounds to at most th: a
// correctly rounded quotient never decreases as x grows.  bound lies within a
// few units in the last place of th * distd; it is found by bisection over the
// bit patterns of the eight doubles around that product (non-negative doubles
// order like their bit patterns), each step one division of the same kind as
// the literal test's.  Returns false where that bracket does not hold (th = 0,
// extreme magnitudes); the trial then runs the literal test.
__device__ __forceinline__ bool pass_bound(double distd, double th, double &bound) {
    if (!(distd >= 1.0) || !(distd < __builtin_inf()) || !(th > 0.0) || !(th < __builtin_inf()))
        return false;
    const double x0 = th * distd;
    if (!(x0 > 0x1p-1000) || !(x0 < 0x1p1000)) return false;
    long long lo = __builtin_bit_cast(long long, x0) - 4;
    long long hi = lo + 8;
    if (!(__builtin_bit_cast(double, lo) / distd <= th) ||
        __builtin_bit_cast(double, hi) / distd <= th)
        return false;
    while (hi - lo > 1) {
        const long long mid = lo + (hi - lo) / 2;
        if (__builtin_bit_cast(double, mid) / distd <= th)
            lo = mid;
        else
            hi = mid;
    }
    bound = __builtin_bit_cast(double, lo);
    return true;
}

// Workgroup LDS of T trials.
template <int T>
struct TrialShared {
    double aa[T], cc[T];  // numerator of each trial's distance
    double bound[T];      // largest |numerator| that passes; -1: invalid trial
    double distd[T];
    int count[T];
    unsigned long long key[T / kWave];
    int literal;  // some trial has no bound: the literal test for all
};

// Adds to sh.count the inliers of the workgroup's trials among the points
// [p0, p1): every lane of the wave takes T / 64 trials, which share each point's
// load (the same address in every lane).
template <int T, bool kLiteral>
__device__ __forceinline__ void count_trials(TrialShared<T> &sh, const double2 *__restrict__ pts,
                                             int p0, int p1, double th, int lane) {
    constexpr int kEach = T / kWave;
    double aa[kEach], cc[kEach], lim[kEach];
    int count[kEach];
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
        const int t = u * kWave + lane;
        aa[u] = sh.aa[t];
        cc[u] = sh.cc[t];
        lim[u] = kLiteral ? sh.distd[t] : sh.bound[t];
        count[u] = 0;
    }
    // A point that takes no part is stored as (NaN, NaN); its distance is NaN and
    // never passes.
    constexpr int kUnroll = kLiteral ? 1 : 8 / kEach;
#pragma unroll kUnroll
    for (int p = p0; p < p1; ++p) {
        const double2 q = pts[p];
#pragma unroll
        for (int u = 0; u < kEach; ++u) {
            const double num = fabs((aa[u] * q.x + q.y) + cc[u]);
            count[u] += (kLiteral ? num / lim[u] <= th : num <= lim[u]) ? 1 : 0;
        }
    }
#pragma unroll
    for (int u = 0; u < kEach; ++u) atomicAdd(&sh.count[u * kWave + lane], count[u]);
}

// Trials [h0, h0 + T) of cluster k by a workgroup: thread t < T draws trial h0 + t
// and fits its line, then the waves share the cluster's points, each counting its
// own for all T trials.  Returns the
// best (count, lowest index) key in every thread (0 when no trial is valid).
// Uniform early return.
template <int T>
__device__ __forceinline__ unsigned long long paper_score(const float *__restrict__ theta, Span sp, int64_t k,
                                          int64_t h0, int32_t n_hyp, uint32_t key0, uint32_t key1,
                                          const double2 *__restrict__ pts, double th,
                                          int32_t *__restrict__ hyp_counts, TrialShared<T> &sh) {
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t h = h0 + tid;
    const bool mine = tid < T && h < n_hyp;
    if (!paper_cluster(sp)) {
        if (hyp_counts != nullptr && mine) hyp_counts[k * n_hyp + h] = 0;
        return 0;
    }
    const int n = (int)sp.n;
    if (tid == 0) sh.literal = 0;
    __syncthreads();
    bool valid = false;
    if (tid < T) {
        Line L;
        L.valid = false;
        double bound = -1.0;
        if (mine) {
            L = trial_line(theta + sp.lo, pts, n, (uint32_t)h, (uint32_t)k, key0, key1);
            valid = L.valid;
            if (valid && !pass_bound(L.distd, th, bound)) sh.literal = 1;
        }
        sh.aa[tid] = valid ? -L.m : 0.0;
        sh.cc[tid] = valid ? -L.c : 0.0;
        sh.bound[tid] = bound;
        sh.distd[tid] = valid ? L.distd : __builtin_nan("");
        sh.count[tid] = 0;
    }
    __syncthreads();
    const int p0 = n * wave / kPaperWaves, p1 = n * (wave + 1) / kPaperWaves;
    if (sh.literal != 0)
        count_trials<T, true>(sh, pts, p0, p1, th, lane);
    else
        count_trials<T, false>(sh, pts, p0, p1, th, lane);
    __syncthreads();
    if (wave < T / kWave) {
        const int count = sh.count[tid];
        if (hyp_counts != nullptr && mine) hyp_counts[k * n_hyp + h] = valid ? count : 0;
        const uint32_t val = valid ? (uint32_t)count + 1u : 0u;
        const uint32_t most = wave_max_u32(val);
        const uint32_t low = ~wave_max_u32(val == most ? ~(uint32_t)h : 0u);
        if (lane == 0)
            sh.key[wave] = most == 0 ? 0ull
                                     : ((unsigned long long)(most - 1u) << 32) | (0xFFFFFFFFull - low);
    }
    __syncthreads();
    unsigned long long key = sh.key[0];
    for (int w = 1; w < T / kWave; ++w) key = sh.key[w] > key ? sh.key[w] : key;
    return key;
}

// Block = (cluster, T trials); blocks of one cluster merge their keys with a 64-bit
// atomic maximum, whose result does not depend on their order.  T = 64 keeps a block
// of the largest cluster short: the blocks run in index order, and with 256 trials
// each the compute unit that happened on several large clusters set the kernel's
// length (512 clusters of 8 to 2048 points, 512 trials, FP64 operations for 14 us:
// 83 us with a thread per trial over all points, 56 us with 256 trials and eight
// waves sharing the points, 45 us this way).
template <int T>
__global__ __launch_bounds__(kPaperBlock) void paper_score_kernel(
    const float *__restrict__ theta, const int32_t *__restrict__ off, int64_t n_points,
    int32_t n_hyp, int32_t blocks_per_cluster, uint32_t key0, uint32_t key1,
    const double2 *__restrict__ xy, const double *__restrict__ thresh,
    unsigned long long *__restrict__ best_key, int32_t *__restrict__ hyp_counts) {
    __shared__ TrialShared<T> sh;
    const int64_t k = blockIdx.x / blocks_per_cluster;
    const int b = (int)(blockIdx.x % blocks_per_cluster);
    const Span sp = cluster_span(off, k, n_points);
    const double2 *pts = paper_cluster(sp) ? xy + sp.lo : xy;
    const unsigned long long key = paper_score<T>(theta, sp, k, (int64_t)b * T, n_hyp, key0, key1,
                                                  pts, thresh[k], hyp_counts, sh);
    if (threadIdx.x == 0 && key != 0) atomicMax(&best_key[k], key);
}

struct PaperOutputs {
    float *vx, *vy, *heading;
    int32_t *n_inliers;
    uint8_t *status;
    int32_t *best;
    uint32_t *bits;
};

__device__ __forceinline__ void paper_failed(const PaperOutputs &o, int64_t k, uint8_t st) {
    const float qnan = __builtin_nanf("");
    o.vx[k] = qnan;
    o.vy[k] = qnan;
    o.heading[k] = qnan;
    o.n_inliers[k] = 0;
    o.status[k] = st;
    if (o.best) o.best[k] = -1;
}

// Refit of cluster k under its kept trial `best` (0: none valid) with
// threshold th (whole workgroup; uniform early returns).
__device__ void paper_refit(const float *__restrict__ theta, const float *__restrict__ vd, Span sp,
                            int64_t k, uint32_t key0, uint32_t key1, const double2 *__restrict__ xy,
                            double th, unsigned long long best, const PaperOutputs &o,
                            double (*s_sum)[5], int *s_cnt) {
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    if (!sp.ok || sp.n < 2 || sp.n > RV_PAPER_MAX_POINTS) {
        if (tid == 0)
            paper_failed(o, k, !sp.ok ? RV_CLUSTER_BAD_OFFSETS
                                      : (sp.n < 2 ? RV_CLUSTER_TOO_FEW_POINTS : RV_CLUSTER_TOO_LARGE));
        return;
    }
    if (best == 0) {
        if (tid == 0) paper_failed(o, k, RV_CLUSTER_ALL_DEGENERATE);
        return;
    }
    const int n = (int)sp.n;
    const uint32_t hbest = 0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull);
    const double2 *pts = xy + sp.lo;
    const Line L = trial_line(theta + sp.lo, pts, n, hbest, (uint32_t)k, key0, key1);
    const int64_t end = sp.lo + sp.n;
    double scc = 0.0, scs = 0.0, sss = 0.0, scv = 0.0, ssv = 0.0;
    int n_in = 0;
    // 64-aligned global blocks of points, so one wave ballot covers two mask words.
    for (int64_t p0 = (sp.lo & ~(int64_t)(kWave - 1)) + (int64_t)wave * kWave; p0 < end;
         p0 += kPaperBlock) {
        const int64_t p = p0 + lane;
        bool inlier = false;
        if (p >= sp.lo && p < end) {
            const double2 q = xy[p];
            if (!__builtin_isnan(q.x) && within(L, q, th)) {
                inlier = true;
                n_in += 1;
                double s, c;
                sincos((double)theta[p], &s, &c);
                const double dv = vd[p];
                scc += c * c;
                scs += c * s;
                sss += s * s;
                scv += c * dv;
                ssv += s * dv;
            }
        }
        if (o.bits != nullptr) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(inlier);
            if (lane == 0) {
                const uint32_t w0 = (uint32_t)m, w1 = (uint32_t)(m >> 32);
                if (w0) atomicOr(&o.bits[p0 >> 5], w0);
                if (w1) atomicOr(&o.bits[(p0 >> 5) + 1], w1);
            }
        }
    }
    scc = wave_sum(scc);
    scs = wave_sum(scs);
    sss = wave_sum(sss);
    scv = wave_sum(scv);
    ssv = wave_sum(ssv);
    n_in = wave_sum_i(n_in);
    if (lane == 0) {
        s_sum[wave][0] = scc;
        s_sum[wave][1] = scs;
        s_sum[wave][2] = sss;
        s_sum[wave][3] = scv;
        s_sum[wave][4] = ssv;
        s_cnt[wave] = n_in;
    }
    __syncthreads();
    if (tid != 0) return;
    scc = s_sum[0][0];
    scs = s_sum[0][1];
    sss = s_sum[0][2];
    scv = s_sum[0][3];
    ssv = s_sum[0][4];
    n_in = s_cnt[0];
    for (int w = 1; w < kPaperWaves; ++w) {
        scc += s_sum[w][0];
        scs += s_sum[w][1];
        sss += s_sum[w][2];
        scv += s_sum[w][3];
        ssv += s_sum[w][4];
        n_in += s_cnt[w];
    }
    o.n_inliers[k] = n_in;
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

__global__ __launch_bounds__(kPaperBlock) void paper_refit_kernel(
    const float *__restrict__ theta, const float *__restrict__ vd, const int32_t *__restrict__ off,
    int64_t n_points, uint32_t key0, uint32_t key1, const double2 *__restrict__ xy,
    const double *__restrict__ thresh, const unsigned long long *__restrict__ best_key,
    PaperOutputs o) {
    __shared__ double s_sum[kPaperWaves][5];
    __shared__ int s_cnt[kPaperWaves];
    const int64_t k = blockIdx.x;
    paper_refit(theta, vd, cluster_span(off, k, n_points), k, key0, key1, xy, thresh[k],
                best_key[k], o, s_sum, s_cnt);
}

// Frames whose clusters each take one workgroup of trials (at most 256), with
// no frame-wide inlier mask requested (its words are shared by neighbouring
// clusters): one launch, a workgroup per cluster, running the threshold step,
// the trials and the refit with the same device functions as the three
// kernels, so every output is theirs bit for bit.  A workgroup reads back only
// the normalised points it wrote itself, after a workgroup barrier.
__global__ __launch_bounds__(kPaperBlock) void paper_frame_kernel(
    const float *__restrict__ theta, const float *__restrict__ vd, const int32_t *__restrict__ off,
    int64_t n_points, int32_t n_hyp, uint32_t key0, uint32_t key1, double2 *__restrict__ xy,
    double *__restrict__ thresh, int32_t *__restrict__ hyp_counts, PaperOutputs o) {
    __shared__ StatsShared sh;
    __shared__ TrialShared<kPaperBlock> s_trials;
    __shared__ double2 s_xy[kPaperBlock];  // normalised points of clusters of <= 256 points
    __shared__ double s_sum[kPaperWaves][5];
    __shared__ int s_cnt[kPaperWaves];
    const int64_t k = blockIdx.x;
    const Span sp = cluster_span(off, k, n_points);
    const double th = paper_stats(theta, vd, sp, k, xy, thresh, sh, s_xy);
    __syncthreads();
    // Trials read the points from LDS where they fit, else from global memory.
    unsigned long long best;
    if (paper_cluster(sp) && sp.n <= kPaperBlock)
        best = paper_score<kPaperBlock>(theta, sp, k, 0, n_hyp, key0, key1, s_xy, th, hyp_counts,
                                        s_trials);
    else
        best = paper_score<kPaperBlock>(theta, sp, k, 0, n_hyp, key0, key1,
                                        paper_cluster(sp) ? xy + sp.lo : xy, th, hyp_counts,
                                        s_trials);
    paper_refit(theta, vd, sp, k, key0, key1, xy, th, best, o, s_sum, s_cnt);
}

constexpr size_t kPaperAlign = 256;
// Frames of at most this many points and clusters take the one-launch path
// (when no inlier mask is requested and n_hyp <= 256).
constexpr int64_t kPaperFrameMaxPoints = 1 << 16;
constexpr int64_t kPaperFrameMaxClusters = 1 << 16;

size_t paper_align(size_t x) { return (x + kPaperAlign - 1) / kPaperAlign * kPaperAlign; }

struct PaperLayout {
    size_t xy, thresh, best_key, total;
};

PaperLayout paper_layout(int64_t n_clusters, int64_t n_points) {
    PaperLayout L;
    size_t at = 0;
    L.xy = at; at = paper_align(at + (size_t)n_points * sizeof(double2));
    L.thresh = at; at = paper_align(at + (size_t)n_clusters * sizeof(double));
    L.best_key = at; at = paper_align(at + (size_t)n_clusters * sizeof(unsigned long long));
    L.total = at;
    return L;
}

}  // namespace

extern "C" {

size_t rv_paper_workspace_bytes(int64_t n_clusters, int64_t n_points, int32_t n_hyp) {
    if (n_clusters < 0 || n_points < 0 || n_hyp < 0) return 0;
    return paper_layout(n_clusters, n_points).total;
}

int rv_estimate_velocity_paper(const float *theta, const float *vd, const int32_t *cluster_offsets,
                               int64_t n_clusters, int64_t n_points, int32_t n_hyp, uint64_t seed,
                               float *vx, float *vy, float *heading, int32_t *n_inliers,
                               uint8_t *status, double *thresh, uint32_t *inlier_bits,
                               int32_t *hyp_counts, int32_t *best_hyp, void *workspace,
                               size_t workspace_bytes, void *stream) {
    g_error[0] = '\0';
    if (n_hyp < 1 || n_hyp > RV_MAX_HYP)
        return fail(RV_ERR_INVALID_ARG, "n_hyp must be in [1, %d]", RV_MAX_HYP);
    if (n_clusters < 0 || n_clusters > INT32_MAX)
        return fail(RV_ERR_INVALID_ARG, "n_clusters must be in [0, 2^31 - 1]");
    if (n_points < 0 || n_points > INT32_MAX)
        return fail(RV_ERR_INVALID_ARG, "n_points must be in [0, 2^31 - 1]");
    if (cluster_offsets == nullptr) return fail(RV_ERR_INVALID_ARG, "cluster_offsets is NULL");
    if (n_points > 0 && (theta == nullptr || vd == nullptr))
        return fail(RV_ERR_INVALID_ARG, "theta or vd is NULL");
    if (n_clusters > 0 && (vx == nullptr || vy == nullptr || heading == nullptr ||
                           n_inliers == nullptr || status == nullptr))
        return fail(RV_ERR_INVALID_ARG, "a required output is NULL");
    const PaperLayout L = paper_layout(n_clusters, n_points);
    if (workspace == nullptr || workspace_bytes < L.total)
        return fail(RV_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", L.total,
                    workspace == nullptr ? (size_t)0 : workspace_bytes);
    if (((uintptr_t)workspace % kPaperAlign) != 0)
        return fail(RV_ERR_WORKSPACE, "workspace must be %zu-byte aligned", kPaperAlign);
    if (n_clusters == 0) return RV_OK;
    const int64_t bpc = ((int64_t)n_hyp + kPaperBlock - 1) / kPaperBlock;
    if (n_clusters * bpc > INT32_MAX) return fail(RV_ERR_INVALID_ARG, "n_clusters * n_hyp too large");
    char *ws = (char *)workspace;
    double2 *xy = (double2 *)(ws + L.xy);
    double *th = thresh != nullptr ? thresh : (double *)(ws + L.thresh);
    unsigned long long *best_key = (unsigned long long *)(ws + L.best_key);
    const uint32_t key0 = (uint32_t)(seed & 0xFFFFFFFFu), key1 = (uint32_t)(seed >> 32);
    hipStream_t st = (hipStream_t)stream;
    PaperOutputs o;
    o.vx = vx;
    o.vy = vy;
    o.heading = heading;
    o.n_inliers = n_inliers;
    o.status = status;
    o.best = best_hyp;
    o.bits = inlier_bits;
    // Stage events (rv_stage_timing): stats and mask clearing, scoring, refit;
    // the one-launch path counts wholly as scoring.
    TimedCall tc;
    const bool timed = take_timed_call(tc);
    if (timed) (void)hipEventRecord(tc.ev[0], st);
    if (inlier_bits == nullptr && n_hyp <= kPaperBlock && n_points <= kPaperFrameMaxPoints &&
        n_clusters <= kPaperFrameMaxClusters) {
        if (timed) (void)hipEventRecord(tc.ev[1], st);
        hipLaunchKernelGGL(paper_frame_kernel, dim3((unsigned)n_clusters), dim3(kPaperBlock), 0, st,
                           theta, vd, cluster_offsets, n_points, n_hyp, key0, key1, xy, th,
                           hyp_counts, o);
        if (timed) {
            (void)hipEventRecord(tc.ev[2], st);
            (void)hipEventRecord(tc.ev[3], st);
            keep_timed_call(tc);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(RV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
        return RV_OK;
    }
    // A mask far larger than the clusters take (most points in none, or in clusters beyond
    // RV_PAPER_MAX_POINTS) gets workgroups that only clear: one cluster in 40M points 143 us a
    // call without them, 19 us with them.
    const int64_t n_words = inlier_bits != nullptr ? (n_points + 31) / 32 : 0;
    const int64_t clearing = (n_words + kClearWords - 1) / kClearWords;
    hipLaunchKernelGGL(paper_stats_kernel,
                       dim3((unsigned)(n_clusters > clearing ? n_clusters : clearing)),
                       dim3(kPaperBlock), 0, st, theta, vd, cluster_offsets, n_clusters, n_points,
                       xy, th, best_key, inlier_bits, n_words);
    if (timed) (void)hipEventRecord(tc.ev[1], st);
    const int64_t bpc64 = ((int64_t)n_hyp + kWave - 1) / kWave;
    // A grid's threads have to stay below 2^32 (HIP refuses it otherwise).
    const bool fine = n_clusters * bpc64 <= (int64_t)UINT32_MAX / kPaperBlock;
    hipLaunchKernelGGL(fine ? paper_score_kernel<kWave> : paper_score_kernel<kPaperBlock>,
                       dim3((unsigned)(n_clusters * (fine ? bpc64 : bpc))), dim3(kPaperBlock), 0, st,
                       theta, cluster_offsets, n_points, n_hyp, (int32_t)(fine ? bpc64 : bpc), key0,
                       key1, (const double2 *)xy, (const double *)th, best_key, hyp_counts);
    if (timed) (void)hipEventRecord(tc.ev[2], st);
    hipLaunchKernelGGL(paper_refit_kernel, dim3((unsigned)n_clusters), dim3(kPaperBlock), 0, st,
                       theta, vd, cluster_offsets, n_points, key0, key1, (const double2 *)xy,
                       (const double *)th, (const unsigned long long *)best_key, o);
    if (timed) {
        (void)hipEventRecord(tc.ev[3], st);
        keep_timed_call(tc);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RV_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    return RV_OK;
}

}  // extern "C"
