// Device helpers shared by the kernels of libfb_amd: the semiring sum in base 2, wave-level reductions, the
// assignment of workgroups to sequences and the progress counters of a launch.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "fb_internal.h"

namespace fb {

namespace {

constexpr float kNegBig = -1.0e30f;   // stands for "no finite term yet"; values below it count as semiring zero
constexpr double kLog2e = 1.4426950408889634074;
constexpr double kLn2 = 0.69314718055994530942;

__device__ __forceinline__ float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float flog2(float x) { return __builtin_amdgcn_logf(x); }

// Maxima of values that are never NaN here: single instructions, without the quieting of
// signalling NaNs that fmaxf() implies.
__device__ __forceinline__ float tmax(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float tmin(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float tmax3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ double tmax(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ double tmax3(double a, double b, double c) { return fmax(fmax(a, b), c); }

// running (+)-sum in base 2: value = m + log2(s); m in the carrier type, s single
template <class T>
__device__ __forceinline__ void lse_add(T &m, float &s, T x)
{
    const float d = (float)(x - m);
    const float e = fexp2(-fabsf(d));
    s = d > 0.0f ? fmaf(s, e, 1.0f) : s + e;
    m = tmax(m, x);
}

// four terms at once: one rescale of the running sum, then plain exponentials
template <class T>
__device__ __forceinline__ void lse_add4(T &m, float &s, T x0, T x1, T x2, T x3)
{
    const T mn = tmax3(tmax3(m, x0, x1), x2, x3);
    const float r = fexp2((float)(m - mn));
    const float e0 = fexp2((float)(x0 - mn)), e1 = fexp2((float)(x1 - mn));
    const float e2 = fexp2((float)(x2 - mn)), e3 = fexp2((float)(x3 - mn));
    s = fmaf(s, r, (e0 + e1) + (e2 + e3));
    m = mn;
}

// four terms whose weights are given as W = 2^w: the running maximum is over the gathered values alone
template <class T>
__device__ __forceinline__ void lse_add4w(T &m, float &s, T g0, T g1, T g2, T g3, float W0, float W1, float W2, float W3)
{
    const T mn = tmax3(tmax3(m, g0, g1), g2, g3);
    const float r = fexp2((float)(m - mn));
    float p = fexp2((float)(g0 - mn)) * W0;
    p = fmaf(fexp2((float)(g1 - mn)), W1, p);
    p = fmaf(fexp2((float)(g2 - mn)), W2, p);
    p = fmaf(fexp2((float)(g3 - mn)), W3, p);
    s = fmaf(s, r, p);
    m = mn;
}

template <class T>
__device__ __forceinline__ void lse_merge(T &m, float &s, T m2, float s2)
{
    const T M = tmax(m, m2);
    s = s * fexp2((float)(m - M)) + s2 * fexp2((float)(m2 - M));
    m = M;
}

// Data-parallel-primitive moves inside rows of 16 lanes, and reads of single lanes, for 32- and 64-bit values.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) { return __uint_as_float(dpp_u<CTRL>(__float_as_uint(v))); }
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint64_t r = (uint64_t)dpp_u<CTRL>((uint32_t)u) | ((uint64_t)dpp_u<CTRL>((uint32_t)(u >> 32)) << 32);
    return __longlong_as_double((long long)r);
}
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v) { return (int)dpp_u<CTRL>((uint32_t)v); }
__device__ __forceinline__ int lane_value(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint64_t r = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l) << 32);
    return __longlong_as_double((long long)r);
}

// v of every lane replaced by op over its aligned group of 2^lg lanes (lg = 1..6, the same in all
// lanes).  Inside a row of 16 lanes: exchanges with the lane whose number differs in one bit
// (the mirror moves equal that exchange once groups of 4 resp. 8 lanes hold one value); across
// rows: the four row results are read into scalars.
template <class V, class Op>
__device__ __forceinline__ V group_all(V v, int lg, int lane, Op op)
{
    v = op(v, dpp_mov<0xB1>(v));                  // quad_perm [1,0,3,2]
    if (lg >= 2) v = op(v, dpp_mov<0x4E>(v));     // quad_perm [2,3,0,1]
    if (lg >= 3) v = op(v, dpp_mov<0x141>(v));    // row_half_mirror
    if (lg >= 4) v = op(v, dpp_mov<0x140>(v));    // row_mirror
    if (lg >= 5) {
        const V lo = op(lane_value(v, 0), lane_value(v, 16)), hi = op(lane_value(v, 32), lane_value(v, 48));
        v = lg == 6 ? op(lo, hi) : (lane < 32 ? lo : hi);
    }
    return v;
}

// (m, s) of every lane replaced by the (+)-sum over its aligned group of 2^lg lanes (all lanes of
// the group end with the same pair): first the maximum, then the sums rescaled to it
template <class T>
__device__ __forceinline__ void group_total(T &m, float &s, int lg, int lane)
{
    const T mg = group_all(m, lg, lane, [](T a, T b) { return tmax(a, b); });
    s = group_all(s * fexp2((float)(m - mg)), lg, lane, [](float a, float b) { return a + b; });
    m = mg;
}

// Tropical semiring: the maximum over the group and the back-pointer of a lane that holds it
// (of the smallest back-pointer among those lanes, so the choice does not depend on timing).
template <class T>
__device__ __forceinline__ void group_best(T &m, int &arg, int lg, int lane)
{
    const T mg = group_all(m, lg, lane, [](T a, T b) { return tmax(a, b); });
    arg = group_all(m == mg ? arg : 0x7fffffff, lg, lane, [](int a, int b) { return min(a, b); });
    m = mg;
}

// reductions over the whole wave; every lane gets the result
template <class T>
__device__ __forceinline__ T wave_max(T v)
{
    return group_all(v, 6, (int)(threadIdx.x & (kWave - 1)), [](T a, T b) { return tmax(a, b); });
}

__device__ __forceinline__ float wave_sum(float v)
{
    return group_all(v, 6, (int)(threadIdx.x & (kWave - 1)), [](float a, float b) { return a + b; });
}

// The largest of a wave's values, in lane 63 (the other lanes hold partial maxima): six maxima that read their neighbour's
// value directly, a lane without one keeping its own.  (wave_max takes a move, a maximum and, across rows, reads into
// scalars instead: 20 instructions and their waits.)
__device__ __forceinline__ float wave_max_last(float v)
{
    asm volatile("s_nop 1\n\t"   // (a value just written may be read from another lane two instructions later)
                 "v_max_f32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\ts_nop 1"
                 : "+v"(v));
    return v;
}

// Sums likewise, always in the same order: of 16 lanes in the last of them, of the wave in lane 63.
__device__ __forceinline__ float row_sum_last(float v)
{
    asm volatile("s_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\ts_nop 1"
                 : "+v"(v));
    return v;
}
__device__ __forceinline__ float wave_sum_last(float v)
{
    v = row_sum_last(v);
    asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\ts_nop 1"
                 : "+v"(v));
    return v;
}

// The word in LDS raised to v, by the lanes that call.  In assembly: for the builtin the compiler first reduces over the
// lanes that are on, in a loop, although a single one is.  The caller's next barrier has to be lds_barrier(), whose wait
// does not depend on what the compiler knows of.
__device__ __forceinline__ void lds_raise(float *word, float v)
{
    asm volatile("ds_max_f32 %0, %1" :: "v"((uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)word), "v"(v) : "memory");
}

// The same for the value that lane 63 holds, in a wave all of whose lanes are on; at: the word's address in LDS.  (A mask
// set and put back instead of a branch around one lane.)
__device__ __forceinline__ void lds_raise_last(uint32_t at, float v)
{
    asm volatile("s_brev_b64 exec, 1\n\tds_max_f32 %0, %1\n\ts_mov_b64 exec, -1" :: "v"(at), "v"(v) : "memory");
}

// A workgroup barrier that waits for what this wave has written to LDS but lets its global loads and stores go on
// (__syncthreads() in a wave that loads straight into LDS waits for all of them).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// f(integral_constant<int, 0>), f(integral_constant<int, 1>), ...: a loop whose counter is a compile-time constant
template <class F, int... I>
__device__ __forceinline__ void unrolled(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// Workgroup -> (sequence, direction).  Workgroups start in the order of their index.  In the large-graph
// kernels (one workgroup fills a compute unit) the longest sequences therefore come first, both
// directions of a sequence side by side: whatever delays the start of a workgroup - a second wave of
// workgroups when there are more than compute units, workgroups of another launch in the way - then
// falls on the sequences that have time to spare.
// (A launch may cover only a range of ranks, P.order then holds the sequences in order of length.)
template <int NW>
__device__ __forceinline__ void resolve_sequence(const RecParams &P, double *lds_raw, int &b, int &which)
{
    constexpr int NT = NW * kWave;
    const int tid = threadIdx.x;
    const int n_launch = P.order ? P.n_launch : P.B;
    b = blockIdx.x % n_launch;
    which = blockIdx.x / n_launch;
    if (NW == kNWShared || P.order) {   // in order of length: both directions of a sequence side by side
        which = blockIdx.x % P.n_dir;
        b = blockIdx.x / P.n_dir;
    }
    if (P.order) {
        b = P.order[P.rank0 + b];
    } else if (NW == kNWShared) {
        const int r = b;   // this workgroup takes the sequence of rank r by length
        int *sel = (int *)lds_raw;
        for (int cand = tid; cand < P.B; cand += NT) {
            const int lc = min(max(P.lengths[cand], 0), P.N);
            int rank = 0;   // sequences that go before cand: the longer ones, and of the equally long the earlier ones
            for (int j = 0; j < P.B; ++j) {
                const int lj = min(max(P.lengths[j], 0), P.N);
                rank += (lj > lc || (lj == lc && j < cand)) ? 1 : 0;
            }
            if (rank == r) *sel = cand;
        }
        __syncthreads();
        b = __builtin_amdgcn_readfirstlane(*sel);
        __syncthreads();   // the word is part of a state buffer from here on
    }
}

// Best path: the frame at which the forward and the backward recursion of a sequence of T > 0 frames meet.  The forward
// one covers frames 0 .. m and the backward one T-1 .. m, side by side.  Row f of the back-pointers joins frame f - 1 and frame f: written by the forward recursion for f <= m, by the
// backward one for f > m.
__device__ __forceinline__ int path_middle(int T) { return (T - 1) >> 1; }

// Progress counter of a launch: everything this workgroup writes is on its way; make it visible device-wide, then count.
// Every wave waits for its own stores first: the barrier alone waits for no global store on this chip, and the fence of
// the thread that counts covers the stores its own wave has made and what has reached the L2 by then - a row that another
// wave still has under way would get there behind the write-back, and a kernel released by the counter on another XCD
// could read what was in memory before.  (One wait per workgroup and launch.)
__device__ __forceinline__ void count_done(const RecParams &P)
{
    if (P.done) {
        const int rank = P.rank0 + (int)blockIdx.x / P.n_dir;   // (launches with counters cover ranks in order)
        int slot = 0;
#pragma unroll
        for (int i = 0; i < kDoneCuts; ++i) slot += rank >= P.done_from[i] ? 1 : 0;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0 && slot > 0) {
            __threadfence();
            atomicAdd(P.done + slot, 1u);
        }
    }
}

}  // namespace

}  // namespace fb
