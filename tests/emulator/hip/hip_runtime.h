// Stands in for the HIP headers when the device code of csrc/rv.hip is compiled for
// the CPU: one workgroup at a time, every lane a fiber, a wave's cross-lane
// operations and the workgroup's barriers as meeting points.  Between two meeting
// points a wave runs alone; which wave runs next is drawn from a seed, so that what
// the hardware's wave order may change shows as a result that depends on the seed.
// A barrier at which the waves stand on different source lines is an error.
// All lanes of a wave take part in every cross-lane operation (as in the kernels).
#pragma once
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <cmath>
#include <functional>
#include <random>
#include <vector>

#include <hip/hip_runtime_api.h>

using std::isfinite;

#define __device__
#define __global__
#define __host__
#define __forceinline__ inline
#define __shared__ static
#define __launch_bounds__(...)
#define amdgpu_waves_per_eu(...) unused
#define __align__(n) __attribute__((aligned(n)))

struct float2 { float x, y; };
struct alignas(16) float4 { float x, y, z, w; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
struct alignas(16) double2 { double x, y; };
inline float2 make_float2(float x, float y) { return {x, y}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
inline double2 make_double2(double x, double y) { return {x, y}; }

struct EmuIndex { uint32_t x; };
static EmuIndex threadIdx, blockIdx, gridDim;

namespace emu {
enum State { kReady, kWaveOp, kBarrier, kDone };
struct Lane {
    ucontext_t ctx;
    std::vector<char> stack;
    State state;
    int line;
};
struct Wave {
    uint64_t slot[64], snap[64];  // operands of the operation being met, and of the last one
};
static std::vector<Lane> lanes;
static std::vector<Wave> waves;
static ucontext_t scheduler;
static const std::function<void()> *body;
static std::function<void()> on_load;  // called before an atomic load (what other workgroups do)

inline void pause(State s, int line) {
    Lane &l = lanes[threadIdx.x];
    l.state = s;
    l.line = line;
    swapcontext(&l.ctx, &scheduler);
}

inline const uint64_t *meet(uint64_t v) {
    const uint32_t t = threadIdx.x;
    waves[t / 64].slot[t % 64] = v;
    pause(kWaveOp, 0);
    return waves[t / 64].snap;
}

inline void start() {
    (*body)();
    lanes[threadIdx.x].state = kDone;
}

inline void fail(const char *what, int a, int b) {
    printf("emulator: %s (%d, %d)\n", what, a, b);
    exit(1);
}

// Runs f as a workgroup of n threads, its waves interleaved as the seed says.
inline void run(int n, uint32_t seed, const std::function<void()> &f) {
    std::mt19937 rng(seed);
    body = &f;
    lanes.resize(n);
    waves.resize(n / 64);
    for (int t = 0; t < n; ++t) {
        Lane &l = lanes[t];
        l.stack.resize(1 << 16);
        l.state = kReady;
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.data();
        l.ctx.uc_stack.ss_size = l.stack.size();
        l.ctx.uc_link = &scheduler;
        makecontext(&l.ctx, start, 0);
    }
    for (;;) {
        std::vector<int> ready;
        int barrier = 0, live = 0;
        for (int w = 0; w < n / 64; ++w) {
            const State s = lanes[w * 64].state;
            if (s == kDone) continue;
            ++live;
            if (s == kBarrier) ++barrier;
            if (s == kReady) ready.push_back(w);
        }
        if (live == 0) return;
        if (barrier == live) {
            int line = -1;
            for (Lane &l : lanes) {
                if (l.state == kDone) continue;
                if (line >= 0 && l.line != line) fail("waves at different barriers, lines", line, l.line);
                line = l.line;
                l.state = kReady;
            }
            continue;
        }
        // A wave that has run ahead keeps its lead now and then, so that another
        // may fall far behind.
        static int last = 0;
        int w = ready[rng() % ready.size()];
        for (int r : ready)
            if (r == last && rng() % 8 != 0) w = r;
        last = w;
        for (int t = w * 64; t < w * 64 + 64; ++t) {
            threadIdx.x = t;
            swapcontext(&scheduler, &lanes[t].ctx);
        }
        const State s = lanes[w * 64].state;
        for (int t = w * 64; t < w * 64 + 64; ++t)
            if (lanes[t].state != s || lanes[t].line != lanes[w * 64].line)
                fail("a wave's lanes have parted, states", s, lanes[t].state);
        if (s == kWaveOp) {
            memcpy(waves[w].snap, waves[w].slot, sizeof waves[w].snap);
            for (int t = w * 64; t < w * 64 + 64; ++t) lanes[t].state = kReady;
        }
    }
}

template <typename T> uint64_t pack(T v) {
    uint64_t u = 0;
    memcpy(&u, &v, sizeof v);
    return u;
}
template <typename T> T unpack(uint64_t u) {
    T v;
    memcpy(&v, &u, sizeof v);
    return v;
}
inline int lane() { return threadIdx.x % 64; }
inline int read_lane(int v, int l) { return unpack<int>(meet(pack(v))[l]); }
inline uint64_t ballot(bool p) {
    const uint64_t *s = meet(p ? 1 : 0);
    uint64_t m = 0;
    for (int l = 0; l < 64; ++l) m |= s[l] << l;
    return m;
}
inline int update_dpp(int old, int v, int ctrl, int rows, int, bool) {
    const uint64_t *s = meet(pack(v));
    const int l = lane(), row = l / 16;
    int from = -1;
    if (ctrl > 0x110 && ctrl < 0x120 && l % 16 >= ctrl - 0x110) from = l - (ctrl - 0x110);
    if (ctrl == 0x142 && row > 0) from = row * 16 - 1;
    if (ctrl == 0x143 && row >= 2) from = 31;
    return ((rows >> row) & 1) && from >= 0 ? unpack<int>(s[from]) : old;
}
inline float med3(float a, float b, float c) {  // with a NaN: the minimum of the others
    if (std::isnan(a)) return fminf(b, c);
    return fmaxf(fminf(a, b), fminf(fmaxf(a, b), c));
}
inline _Float16 half_rtz(float f) {
    _Float16 h = (_Float16)f;
    if (fabsf((float)h) > fabsf(f)) h = unpack<_Float16>(pack(h) - 1);
    return h;
}
inline uint32_t pkrtz(float a, float b) {
    return (uint32_t)pack(half_rtz(a)) | (uint32_t)pack(half_rtz(b)) << 16;
}
inline float dot2(uint32_t a, uint32_t b, float c) {
    const float p = (float)unpack<_Float16>(a) * (float)unpack<_Float16>(b);
    return p + (float)unpack<_Float16>(a >> 16) * (float)unpack<_Float16>(b >> 16) + c;
}
template <typename T> T atomic_load(const T *p) {
    if (on_load) on_load();
    return *p;
}
// Four rows of the FP16 form (inline assembly in the kernel).
inline uint32_t dot_count4(const uint32_t (&c)[4], const float (&w)[4], uint32_t nd, float t) {
    uint32_t n = 0;
    for (int i = 0; i < 4; ++i) n += __builtin_popcountll(ballot(fabsf(dot2(c[i], nd, w[i])) < t));
    return n;
}
}  // namespace emu

inline int amdgcn_writelane(int value, int lane, int old) { return emu::lane() == lane ? value : old; }
template <typename T> T __shfl_xor(T v, int o, int) { return emu::unpack<T>(emu::meet(emu::pack(v))[emu::lane() ^ o]); }
template <typename T> T __shfl_up(T v, int d, int width) {
    const uint64_t *s = emu::meet(emu::pack(v));
    const int l = emu::lane();
    return emu::unpack<T>(s[l % width >= d ? l - d : l]);
}
template <typename T, typename U> T atomicAdd(T *p, U v) { const T old = *p; *p += v; return old; }
template <typename T, typename U> T atomicOr(T *p, U v) { const T old = *p; *p |= v; return old; }
template <typename T, typename U> T atomicMax(T *p, U v) { const T old = *p; if (v > *p) *p = v; return old; }

#define __syncthreads() emu::pause(emu::kBarrier, __LINE__)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) emu::atomic_load(p)
#define __builtin_amdgcn_readfirstlane(v) emu::read_lane(v, 0)
#define __builtin_amdgcn_readlane(v, l) emu::read_lane(v, l)
#define __builtin_amdgcn_ballot_w64(p) emu::ballot(p)
#define __builtin_amdgcn_update_dpp emu::update_dpp
#define __builtin_amdgcn_mbcnt_lo(m, c) ((c) + (uint32_t)__builtin_popcountll((m) & ((1ull << emu::lane()) - 1)))
#define __builtin_amdgcn_mbcnt_hi(m, c) \
    ((c) + (uint32_t)__builtin_popcountll(((uint64_t)(m) << 32) & ((1ull << emu::lane()) - 1)))
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __builtin_amdgcn_bitop3_b32(a, b, c, table) ((a) ^ (b) ^ (c))
#define __builtin_amdgcn_fmed3f(a, b, c) emu::med3(a, b, c)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsqf(x) (1.0f / sqrtf(x))
#define __builtin_amdgcn_sqrtf(x) sqrtf(x)
#define __builtin_amdgcn_cvt_pkrtz(a, b) emu::pkrtz(a, b)
