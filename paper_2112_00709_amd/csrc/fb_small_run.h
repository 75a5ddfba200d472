// The recursions of small (sub-)graphs in the log semifield: what a workgroup does for one (sequence, direction), for the
// kernel of fb_small.hip, where the reasons are, and as what a run of fb_small_linear.hip that leaves its range is done over by.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "fb_device.h"
#include "fb_internal.h"

namespace fb {

namespace {

constexpr double kZero = -1.0e36, kZeroOut = -1.0e30;

__device__ __forceinline__ bool is_zero(double v) { return v <= kZeroOut; }   // (false for a NaN)

// an emission in log2 units, zero-bar as kZero; a NaN stays one
__device__ __forceinline__ double emitted(float e) { return (double)(e < (float)kZero ? (float)kZero : e) * kLog2e; }

template <int NC, int R, int WRITERS = NC == 1 ? 2 : 4>
struct SmallShape {
    static constexpr int NIO = WRITERS;                                  // waves that write rows out
    static constexpr int KS = NC * R * kWave < kSmallStates ? NC * R * kWave : kSmallStates;   // states at most
    static constexpr int XS = KS + 2;                                    // entries of a row in LDS; entry KS takes what nobody wants
    static constexpr int RPB = NC == 1 ? 8 : 1;                          // frames between two barriers
    static constexpr int RB = 2 * RPB;                                   // rows of the ring
    static constexpr int kAhead = NC == 1 ? 16 : R >= 3 ? 4 : 8;         // frames whose emissions are asked for at a time
    static constexpr int UIO = KS / kWave;                               // states per lane of a writing wave
    static_assert(kAhead % RB == 0, "the ring row of an unrolled step is a constant");
    // x ring, ring of the rows before the emission (backward), back-pointer ring (best path), reduction scratch, two words
    // per computing wave
    static constexpr size_t lds_bytes(bool backward, bool tropical)
    {
        return (size_t)RB * XS * 8 * (backward && !tropical ? 2 : 1) + (tropical ? (size_t)RB * XS * 2 : 0) + 8 * (2 * (size_t)NC) +
               4 * (2 * (size_t)NC) + 16;
    }
};

// The launch's parameters where the kernel finds them, and what they point to.  (Spelled out for functions that are not part of the
// kernel, to which a pointer read from memory might point anywhere: an access through such a one counts as one to LDS too, so a barrier waits
// for every load and store, and every store might change a parameter.)
typedef const __attribute__((address_space(4))) RecParams LaunchParams;
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T *in_global(T *p)
{
    return (__attribute__((address_space(1))) T *)(uintptr_t)p;
}

// What a finite value is larger than kLarge in size by, as a number to take the maximum of: the size's bits, moved so that
// infinities and NaN wrap round to small ones.
constexpr uint32_t kLargeBits = (0x47800000u << 1) + 0x01000000u;   // ... that number of kLarge = 65536
__device__ __forceinline__ uint32_t size_bits(float x) { return (__float_as_uint(x) << 1) + 0x01000000u; }

// the larger of two values that are never NaN: one instruction, without the quieting of NaNs that fmax() implies
__device__ __forceinline__ double dmax(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// A lane's rows of the next vector from the gathered entries g, weights w and emissions ed (log2 units): into x, and into
// pre before the emission (backward) or bp, where it came from (best path), all at the rows' places tg.
template <int R, int TM, bool TROP, bool BWD>
__device__ __forceinline__ void small_fold(const double (&g)[R][TM], const double (&w)[R][TM], const uint32_t (&so)[R][TM], const double (&ed)[R],
                                           const int (&lg)[R], int lane, const uint32_t (&tg)[R], char *x_row, char *pre_row, char *bp_row)
{
#pragma unroll
    for (int j = 0; j < R; ++j) {
        double m;
        if constexpr (TROP) {
            uint32_t arg = so[j][0];
            m = g[j][0] + w[j][0];
#pragma unroll
            for (int t = 1; t < TM; ++t) {                  // (the first of equal terms)
                const double x = g[j][t] + w[j][t];
                uint32_t from = so[j][t];
                asm("" : "+v"(from));                       // (or the compiler may choose between two addresses of so, which then is memory)
                if (x > m) { m = x; arg = from; }
            }
            if (TM > 2 && lg[j]) {
                int ai = (int)arg;
                group_best(m, ai, lg[j], lane);
                arg = (uint32_t)ai;
            }
            *(double *)(x_row + tg[j]) = dmax(m + ed[j], -INFINITY);
            *(uint16_t *)(bp_row + (tg[j] >> 2)) = (uint16_t)(arg >> 3);
        } else {
            float l;
            if constexpr (TM == 2) {                        // two terms: the larger + log2(1 + 2^-|difference|)
                const double x0 = g[j][0] + w[j][0], x1 = g[j][1] + w[j][1];
                m = dmax(x0, x1);
                l = flog2(1.0f + fexp2(-fabsf((float)(x0 - x1))));
            } else {
                double x[TM];
#pragma unroll
                for (int t = 0; t < TM; ++t) x[t] = g[j][t] + w[j][t];
                m = dmax(dmax(x[0], x[1]), dmax(x[2], x[3]));
                float s = (fexp2((float)(x[0] - m)) + fexp2((float)(x[1] - m))) + (fexp2((float)(x[2] - m)) + fexp2((float)(x[3] - m)));
                if (lg[j]) group_total(m, s, lg[j], lane);
                l = flog2(s);
            }
            *(double *)(x_row + tg[j]) = (m + ed[j]) + (double)l;
            if constexpr (BWD) *(double *)(pre_row + tg[j]) = m + (double)l;
        }
    }
}

// The plain form of a (sequence, direction) run, by the whole workgroup, for sequences with large emissions: step by step, the
// largest entry of the previous vector taken off at every step, rows stored by the waves that compute them once their
// largest entry is known.  Returns what has been taken off in all.  A function of its own that reads the launch's parameters
// anew: as part of the kernel it cost calls that never need it 1 to 4 % (registers, and code to fetch at every launch).
template <int NC, int R, int TM, bool TROP>
__device__ __attribute__((noinline)) double small_plain(__attribute__((address_space(3))) double *lds_raw, uint64_t args, int b_, int which_, int Tn_, int Ts_)
{
    double *const xr = (double *)lds_raw;
    // (arguments arrive in vector registers; args: where the launch's parameters are, which only the kernel itself can tell)
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int b = uniform(b_), which = uniform(which_), Tn = uniform(Tn_), Ts = uniform(Ts_);
    args = (uint64_t)(uint32_t)uniform((int)(uint32_t)args) | (uint64_t)(uint32_t)uniform((int)(uint32_t)(args >> 32)) << 32;
    using S = SmallShape<NC, R>;
    constexpr int XS = S::XS, RB = S::RB;
    constexpr uint32_t kRow = XS * 8;
    constexpr double kNone = TROP ? -INFINITY : kZero;
    const RecParams &P = *(const RecParams *)args;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // (rows of the first attempt arrive before these are stored)
    lds_barrier();
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= NC) {
        for (int i = 0; i < Ts; ++i) lds_barrier();
        return 0.0;
    }
    const RecDir &D = P.dir[which];
    const bool bwd = D.backward != 0, pre = bwd && !TROP;
    const SmallSub sd = D.small.sub[P.shared ? 0 : b];
    double *pr = xr + (size_t)RB * XS;
    uint16_t *bpr = (uint16_t *)(pr + (pre ? (size_t)RB * XS : 0));
    char *const lds = (char *)xr;
    const size_t out_ld = P.shared ? (size_t)(D.out_ld ? D.out_ld : sd.K) : (size_t)P.Ktot;
    const size_t out_at = P.shared ? (size_t)b * P.N * out_ld : (size_t)sd.k0;
    auto frame = [&](int i) { return bwd ? Tn - 1 - i : i; };
    uint32_t so[R][TM], tg[R], po[R];
    double w[R][TM];
    int lg[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int s = wave + j * NC;
        const bool have = s < sd.n_slice;
        const size_t at = (size_t)(sd.slice0 + (have ? s : 0));
        const uint32_t row = have ? D.small.rows[at * kWave + lane] : kSmallNoRow;
        lg[j] = have ? __builtin_amdgcn_readfirstlane(D.small.lg[at]) : 0;
        tg[j] = row == kSmallNoRow ? (uint32_t)S::KS * 8u : row * 8u;
        po[j] = (uint32_t)P.pdf[sd.k0 + (row == kSmallNoRow ? 0 : (int)row)] * 4u;
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            const Arc a = D.small.arcs[(at * TM + t) * kWave + lane];
            so[j][t] = (uint32_t)a.src;
            w[j][t] = have ? dmax((double)a.w, kNone) : kNone;
        }
    }
    // (address spaces spelled out: a generic store would count as an access to LDS too, and a barrier would wait for it)
    typedef __attribute__((address_space(1))) char *gptr;
    auto global = [](const void *p) { return (gptr)(uintptr_t)p; };
    typedef __attribute__((address_space(1))) float gf;
    typedef __attribute__((address_space(1))) double gd;
    typedef __attribute__((address_space(1))) uint16_t gu16;
    float e[R], e1[R];                                      // emissions of the step in hand, and of the next
    auto emissions = [&](int i, float(&to)[R]) {
        const gptr row = global(P.emis + ((size_t)b * P.N + (size_t)frame(i)) * P.D);
#pragma unroll
        for (int j = 0; j < R; ++j) to[j] = *(const gf *)(row + po[j]);
    };
    auto largest = [&](const double *row) {                 // (0 if it is zero-bar)
        double mx = -INFINITY;
        for (int k = lane; k < sd.K; k += kWave) mx = dmax(mx, row[k]);
        mx = wave_max(mx);
        return mx == -INFINITY || (!TROP && is_zero(mx)) ? 0.0 : mx;
    };
    emissions(0, e);
    if (Ts > 1) emissions(1, e1);
    const gptr out = global(D.out), bp = global(D.bp), off = global(D.off), cum = global(D.cum);
    const bool carrier = D.out_carrier != 0, has_out = D.out != nullptr, has_bp = TROP && D.bp != nullptr;
    const float scale = D.out_scale;
    const int N = P.N;
    const bool shared = P.shared != 0;
    const int64_t bp_ld = D.bp_ld;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const double s = tg[j] != (uint32_t)S::KS * 8u ? (double)D.bound[sd.k0 + (int)(tg[j] >> 3)] : kNone;
        *(double *)(lds + tg[j]) = TROP ? dmax(s + (bwd && Ts == 1 ? 0.0 : (double)e[j] * kLog2e), kNone) : dmax(s, kNone) + emitted(e[j]);
        if (pre) *(double *)((char *)pr + tg[j]) = s;
    }
    lds_barrier();
    double csum = 0.0;
#pragma unroll 1
    for (int i = 1;; ++i) {
        const uint32_t cur = (uint32_t)((i - 1) % RB) * kRow, nxt = (uint32_t)(i % RB) * kRow;
#pragma unroll
        for (int j = 0; j < R; ++j) e[j] = e1[j];
        if (i + 1 < Ts) emissions(i + 1, e1);
        const double c = largest((const double *)(lds + cur));
        const double *row = (const double *)((pre ? (const char *)pr : lds) + cur);   // row i - 1 -> global memory
        const double mr = pre ? largest(row) : c;
        const int f = frame(i - 1);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (tg[j] == (uint32_t)S::KS * 8u) continue;
            const size_t k = tg[j] >> 3, at = out_at + (size_t)f * out_ld + k;
            const double v = row[k];
            if (has_out && carrier) ((gd *)out)[at] = is_zero(v) ? -INFINITY : v;
            else if (has_out) ((gf *)out)[at] = is_zero(v) ? -INFINITY : (float)(v - mr) * scale;
            if (has_bp && i > 1) {
                const int r = bwd ? f + 1 : f;              // (path_middle)
                ((gu16 *)bp)[(shared ? ((size_t)b * N + r) * bp_ld : (size_t)r * bp_ld + sd.k0) + k] = bpr[(tg[j] >> 3) + cur / 8];
            }
        }
        if (wave == 0 && lane == 0) {
            if (D.off && !(has_out && carrier)) ((gd *)off)[(size_t)b * N + f] = (mr + csum) * (double)scale;
            if (D.cum) ((gf *)cum)[(size_t)b * N + f] = (float)csum;
        }
        if (i >= Ts) return csum;
        csum += c;
        double g[R][TM], ed[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {                       // (off the entries: a sum with a weight would lose the weight first)
#pragma unroll
            for (int t = 0; t < TM; ++t) {
                const double x = *(const double *)(lds + so[j][t] + cur);
                g[j][t] = !TROP && is_zero(x) ? kZero : x - c;
            }
            ed[j] = !TROP ? emitted(e[j]) : bwd && i == Ts - 1 ? 0.0 : (double)e[j] * kLog2e;
        }
        if (bwd) small_fold<R, TM, TROP, true>(g, w, so, ed, lg, lane, tg, lds + nxt, (char *)pr + nxt, (char *)bpr + nxt / 4);
        else small_fold<R, TM, TROP, false>(g, w, so, ed, lg, lane, tg, lds + nxt, nullptr, (char *)bpr + nxt / 4);
        lds_barrier();
    }
}

// The rows of the frames behind the sequence's end, by NT threads.
template <int NT, class F, class D64>
__device__ __forceinline__ void small_pad(bool fill, F out_f, D64 off_seq, size_t out_ld, int Tn, int N, int K)
{
    if (!fill) return;
    const int tid = threadIdx.x;
    if (out_f)
        for (int f = Tn; f < N; ++f)
            for (int k = tid; k < K; k += NT) out_f[(size_t)f * out_ld + k] = -INFINITY;
    if (off_seq)
        for (int f = Tn + tid; f < N; f += NT) off_seq[f] = 0.0;
}

// A (sequence, direction) run by the whole workgroup of NC + NIO waves, its padded frames included; args: where the launch's parameters
// are in memory (P is them); plain: in the plain form at once.
template <int NC, int R, int TM, bool TROP, int NIO, class PARAMS>
__device__ __forceinline__ void small_run(PARAMS &P, uint64_t args, double *lds_raw, const int b, const int which, const bool plain = false)
{
    using S = SmallShape<NC, R, NIO>;
    constexpr int XS = S::XS, RPB = S::RPB, RB = S::RB, A = S::kAhead;
    constexpr double kNone = TROP ? -INFINITY : kZero;      // zero-bar
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const auto &D = P.dir[which];
    const bool bwd = D.backward != 0, pre = bwd && !TROP;   // pre: rows leave before the emission is applied
    const SmallSub sd = D.small.sub[P.shared ? 0 : b];
    const int K = sd.K, k0 = sd.k0;
    const int Tn = min(max(in_global(P.lengths)[b], 0), P.N);
    const int mid = path_middle(Tn);
    const int Ts = Tn > 0 && TROP ? (bwd ? Tn - mid : mid + 1) : Tn;   // frames this direction visits
    auto frame = [&](int i) { return bwd ? Tn - 1 - i : i; };

    double *xr = lds_raw;                                   // [RB][XS]
    double *pr = xr + (size_t)RB * XS;                      // [RB][XS], backward only
    uint16_t *bpr = (uint16_t *)(pr + (pre ? (size_t)RB * XS : 0));   // [RB][XS], best path only
    double *fin = (double *)(bpr + (TROP ? (size_t)RB * XS : 0));     // [NC] + [NC] last reduction
    uint32_t *large_w = (uint32_t *)(fin + 2 * NC);         // [NC] large emissions among a wave's first ones, [NC] ... among all
    double csum = 0.0;                                      // computing waves: what has been taken off the vector

    const size_t out_ld = P.shared ? (size_t)(D.out_ld ? D.out_ld : K) : (size_t)P.Ktot;
    const size_t out_at = P.shared ? (size_t)b * P.N * out_ld : (size_t)k0;
    const auto out_f = in_global((D.out && !D.out_carrier) ? (float *)D.out + out_at : nullptr);
    const auto out_t = in_global((D.out && D.out_carrier) ? (double *)D.out + out_at : nullptr);
    const auto off_seq = in_global(D.off ? D.off + (size_t)b * P.N : nullptr);
    const int n_bar = (Ts - 1 + RPB - 1) / RPB;             // blocks of rows behind the first one
    const bool shifted = !out_t && (out_f || off_seq);      // rows leave without their largest entry
    // (behind a barrier) whether a wave has told of large emissions
    auto told = [&](int at) -> bool { return __any(large_w[at + (lane & (NC - 1))] != 0u); };

    bool again = false;                                     // (uniform) the sequence is to be done over
    if (Tn > 0 && wave < NC) {
        // ---- computing waves
        uint32_t so[R][TM], tg[R];
        double w[R][TM];
        uint32_t po[R];                                     // the lane's place in a row of emissions, bytes
        int lg[R];
        char *const lds = (char *)lds_raw;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int s = wave + j * NC;
            const bool have = s < sd.n_slice;               // (a slice that is not there: every lane adds up nothing)
            const size_t at = (size_t)(sd.slice0 + (have ? s : 0));
            const uint32_t row = have ? in_global(D.small.rows)[at * kWave + lane] : kSmallNoRow;
            lg[j] = have ? __builtin_amdgcn_readfirstlane(in_global(D.small.lg)[at]) : 0;
            tg[j] = row == kSmallNoRow ? (uint32_t)S::KS * 8u : row * 8u;
            po[j] = (uint32_t)in_global(P.pdf)[k0 + (row == kSmallNoRow ? 0 : (int)row)] * 4u;
#pragma unroll
            for (int t = 0; t < TM; ++t) {
                const auto a = in_global(D.small.arcs) + (at * TM + t) * kWave + lane;
                so[j][t] = (uint32_t)a->src;
                w[j][t] = have ? dmax((double)a->w, kNone) : kNone;
            }
        }
        // the row of emissions to ask for next (uniform): the frames in order of the steps, the last one again behind the end
        const ptrdiff_t em_step = bwd ? -(ptrdiff_t)P.D : (ptrdiff_t)P.D;
        auto em_row = in_global(P.emis + ((size_t)b * P.N + (size_t)frame(0)) * P.D);
        int em_left = Ts - 1;
        auto next_em = [&]() {
            em_row += em_left > 0 ? em_step : 0;
            --em_left;
        };
        typedef const __attribute__((address_space(1))) char gchar;
        typedef const __attribute__((address_space(1))) float gfloat;
        auto emission = [&](int j) { return *(gfloat *)((gchar *)em_row + po[j]); };
        auto ask = [&](float(&to)[R][A]) __attribute__((always_inline)) {   // the next A frames' emissions
#pragma unroll
            for (int a = 0; a < A; ++a) {
#pragma unroll
                for (int j = 0; j < R; ++j) to[j][a] = emission(j);
                next_em();
            }
        };
        uint32_t size = plain ? ~0u : D.small.large;        // the largest of size_bits() so far
        auto tell = [&](int at) {
            const bool any = __any(size > kLargeBits);
            if (lane == 0) large_w[at + wave] = any ? 1u : 0u;
        };
        float e[R][A];
        {   // first frame: start weight (x) emission
            float e0[R];
#pragma unroll
            for (int j = 0; j < R; ++j) e0[j] = emission(j);
            next_em();
            ask(e);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const bool real = tg[j] != (uint32_t)S::KS * 8u;
                const double s = real ? (double)in_global(D.bound)[k0 + (int)(tg[j] >> 3)] : kNone;
                // (a best path's backward recursion ends before the emission of its last frame, which may be this one)
                *(double *)(lds + tg[j]) = TROP ? dmax(s + (bwd && Ts == 1 ? 0.0 : (double)e0[j] * kLog2e), kNone) : dmax(s, kNone) + emitted(e0[j]);
                if (pre) *(double *)((char *)pr + tg[j]) = s;
                size = max(size, size_bits(e0[j]));
            }
        }
        tell(0);
        lds_barrier();
        constexpr uint32_t kRow = XS * 8;
        // step i0 + a, a < A a constant
        auto step = [&](auto ac, auto bwd_c, int i0) __attribute__((always_inline)) {
            constexpr int a = decltype(ac)::value;
            constexpr bool kBwd = decltype(bwd_c)::value;
            constexpr uint32_t cur = (a % RB) * kRow, nxt = ((a + 1) % RB) * kRow;
            double g[R][TM];
#pragma unroll
            for (int j = 0; j < R; ++j)
#pragma unroll
                for (int t = 0; t < TM; ++t) g[j][t] = *(const double *)(lds + so[j][t] + cur);
            double ed[R];
#pragma unroll
            for (int j = 0; j < R; ++j) {                   // (best path: see above)
                ed[j] = !TROP ? emitted(e[j][a]) : kBwd && i0 + a == Ts - 1 ? 0.0 : (double)e[j][a] * kLog2e;
                size = max(size, size_bits(e[j][a]));
            }
            if (NC == 1 && !TROP) __builtin_amdgcn_sched_barrier(0);   // (that is done while the gathers are under way)
            small_fold<R, TM, TROP, kBwd>(g, w, so, ed, lg, lane, tg, lds + nxt, (char *)pr + nxt, (char *)bpr + nxt / 4);
            if constexpr ((a + 1) % RPB == 0) lds_barrier();
            __builtin_amdgcn_sched_barrier(0);              // (what belongs to a step stays in it)
        };
        // Groups of A steps without a branch between them; a group's emissions are asked for all at once when the group
        // before it begins.  (Asked for one step's at a time, in the place of those just used, they end up in registers of
        // their own that the compiler moves into place at the end of the group - and has to wait for there.)
        auto all_steps = [&](auto bwd_c) __attribute__((always_inline)) {
            constexpr auto kA = std::make_integer_sequence<int, A>{};
            int i0 = 1;
            for (; i0 + A <= Ts; i0 += A) {
                float ahead[R][A];
                ask(ahead);
                __builtin_amdgcn_sched_barrier(0);
                unrolled([&](auto ac) __attribute__((always_inline)) { step(ac, bwd_c, i0); }, kA);
#pragma unroll
                for (int j = 0; j < R; ++j)
#pragma unroll
                    for (int a = 0; a < A; ++a) e[j][a] = ahead[j][a];
            }
            unrolled([&](auto ac) __attribute__((always_inline)) {
                if (i0 + decltype(ac)::value < Ts) step(ac, bwd_c, i0);
            }, kA);
        };
        again = told(0);
        if (!again) {
            if (bwd) all_steps(std::true_type{});
            else all_steps(std::false_type{});
            if ((Ts - 1) % RPB != 0) lds_barrier();         // the last block's rows
            tell(NC);
            lds_barrier();
            again = told(NC);
        }
    } else if (Tn > 0) {
        // ---- writing waves: a row is one wave's, the rows go round the waves
        const int q = wave - NC;
        const double *rows = pre ? pr : xr;
        const double scale = (double)D.out_scale;
        struct Row { double v[TROP ? 1 : S::UIO]; uint16_t p[TROP ? S::UIO : 1]; double c; };   // (a best path's vectors do not leave)
        // the lane's u-th state; lanes behind the last state take that one again (and store the same value to the same place:
        // no lane has to be masked out)
        auto at = [&](int u) { return min(u * kWave + lane, K - 1); };
        auto fetch = [&](int i, Row &r) __attribute__((always_inline)) {   // row i of the ring -> registers
            if constexpr (TROP) {
                const uint16_t *srow = bpr + (size_t)(i % RB) * XS;
#pragma unroll
                for (int u = 0; u < S::UIO; ++u) r.p[u] = srow[at(u)];
            } else {
                const double *row = rows + (size_t)(i % RB) * XS;
#pragma unroll
                for (int u = 0; u < S::UIO; ++u) r.v[u] = row[at(u)];
            }
        };
        auto take_shift = [&](Row &r) __attribute__((always_inline)) {     // the row's largest entry (any number near it serves)
            if (TROP || !shifted) return;
            float mx = -INFINITY;
#pragma unroll
            for (int u = 0; u < S::UIO; ++u)
                if (u * kWave < K) mx = tmax(mx, (float)r.v[u]);
            mx = wave_max(mx);
            r.c = (double)mx > kZeroOut ? (double)mx : 0.0;
        };
        auto emit = [&](int i, const Row &r, auto u0, auto u1) __attribute__((always_inline)) {   // states u0 * 64 .. u1 * 64 of row i -> global memory
            const int f = frame(i);
            if constexpr (TROP) {
                if (i > 0) {
                    const int row = bwd ? f + 1 : f;         // (path_middle)
                    const auto orow = in_global(D.bp) + (P.shared ? ((size_t)b * P.N + row) * D.bp_ld : (size_t)row * D.bp_ld + k0);
#pragma unroll
                    for (int u = u0; u < u1; ++u)
                        if (u * kWave < K) orow[at(u)] = r.p[u];
                }
            } else {
                if (shifted) {
                    if (out_f) {
                        const auto orow = out_f + (size_t)f * out_ld;
#pragma unroll
                        for (int u = u0; u < u1; ++u)
                            if (u * kWave < K) orow[at(u)] = is_zero(r.v[u]) ? -INFINITY : (float)(r.v[u] - r.c) * D.out_scale;
                    }
                    if (off_seq && u0 == 0 && lane == 0) off_seq[f] = r.c * scale;
                } else if (out_t) {
                    const auto orow = out_t + (size_t)f * out_ld;
#pragma unroll
                    for (int u = u0; u < u1; ++u)
                        if (u * kWave < K) orow[at(u)] = is_zero(r.v[u]) ? -INFINITY : r.v[u];
                }
                if (D.cum && u0 == 0 && lane == 0) in_global(D.cum)[(size_t)b * P.N + f] = 0.0f;   // (carrier rows are not shifted)
            }
        };
        using N0 = std::integral_constant<int, 0>;
        using NH = std::integral_constant<int, (S::UIO + 1) / 2>;
        using NU = std::integral_constant<int, S::UIO>;
        // behind the barrier of block n: whether that was the last one and the sequence is to be done over
        auto over = [&](int n) -> bool {
            if (n < n_bar) return false;
            lds_barrier();
            return told(NC);
        };
        const bool any_row = TROP ? D.bp != nullptr : shifted || out_t || D.cum;
        if constexpr (NC == 1) {
            // the rows of a block: a wave's share of them all read, then all maxima (independent chains), then all stored
            constexpr auto kMine = std::make_integer_sequence<int, RPB / NIO>{};
            auto block = [&](int i0, int cnt) __attribute__((always_inline)) {
                Row r[RPB / NIO];
                unrolled([&](auto x) __attribute__((always_inline)) { fetch(i0 + x * NIO + q, r[x]); }, kMine);   // (rows behind cnt: read and not used)
                unrolled([&](auto x) __attribute__((always_inline)) { take_shift(r[x]); }, kMine);
                unrolled([&](auto x) __attribute__((always_inline)) {
                    if (x * NIO + q < cnt) emit(i0 + x * NIO + q, r[x], N0{}, NU{});
                }, kMine);
            };
            lds_barrier();
            again = told(0) || over(0);
            if (any_row && !again) block(0, 1);
            for (int n = 1; n <= n_bar && !again; ++n) {
                lds_barrier();                              // block n is in the ring
                again = over(n);
                if (any_row && !again) block((n - 1) * RPB + 1, min(RPB, Ts - 1 - (n - 1) * RPB));
            }
        } else {
            // a wave's row takes it four steps: read (it is gone two steps later), maximum, first half stored, second half
            static_assert(NIO == 4 || NIO == 8, "stages of a row");
            Row r;
            auto stage = [&](int s, int i) __attribute__((always_inline)) {
                if (s == 0) fetch(i, r);
                else if (s == 1) take_shift(r);
                else if (s == 2) emit(i, r, N0{}, NH{});
                else emit(i, r, NH{}, NU{});
            };
            lds_barrier();
            again = told(0);
            if (!again) {
                if (any_row && q == 0) stage(0, 0);
                for (int n = 1; n <= n_bar; ++n) {
                    lds_barrier();                          // row n is in the ring
                    const int s = (n - q) & (NIO - 1);
                    if (any_row && s < 4 && n >= s) stage(s, n - s);
                }
                lds_barrier();
                again = told(NC);
            }
            const int s = (n_bar - q) & (NIO - 1);
            if (any_row && n_bar >= s && !again)
                for (int t = s + 1; t < 4; ++t) stage(t, n_bar - s);
        }
    }
    if (__builtin_expect(again, 0)) csum = small_plain<NC, R, TM, TROP>((__attribute__((address_space(3))) double *)lds_raw, args,
                                                                             b, which, Tn, Ts);

    if (Tn > 0) {
        const double *xl = xr + (size_t)((Ts - 1) % RB) * XS;
        if constexpr (TROP) {
            // ---- the last vector, for the kernel that joins the two halves
            const auto mrow = in_global((double *)D.mid) + (size_t)b * D.mid_ld;
            double c = 0.0;
            if (__builtin_expect(again, 0)) {               // (without its largest entry: the other half's vector is added to it)
                c = -INFINITY;
                for (int k = lane; k < K; k += kWave) c = dmax(c, xl[k]);
                c = wave_max(c);
                c = c == -INFINITY ? 0.0 : c;
            }
            if (wave < NC)
                for (int k = wave * kWave + lane; k < K; k += NC * kWave) mrow[k] = xl[k] - c;
            if (threadIdx.x == 0) D.mid_off[b] = csum + c;
        } else {
            // ---- log Z from the last vector and the end weights, by the computing waves
            if (wave < NC) {
                double m = (double)kNegBig;
                float s = 0.0f;
                for (int k = wave * kWave + lane; k < K; k += NC * kWave) lse_add(m, s, xl[k] + (double)in_global(D.obound)[k0 + k]);
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) lse_merge(m, s, __shfl_xor(m, o, 64), __shfl_xor(s, o, 64));
                if (lane == 0) { fin[wave] = m; fin[NC + wave] = (double)s; }
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                double m = fin[0];
                float s = (float)fin[NC];
                for (int v = 1; v < NC; ++v) lse_merge(m, s, fin[v], (float)fin[NC + v]);
                if (D.logz) D.logz[b] = is_zero(m) && s == s ? -INFINITY : ((m + (double)flog2(s)) + csum) * kLn2;   // (a NaN is in s)
            }
        }
    } else if (threadIdx.x == 0 && D.logz) {
        D.logz[b] = -INFINITY;
    }

    small_pad<(NC + NIO) * kWave>(D.fill_pad != 0, out_f, off_seq, out_ld, Tn, P.N, K);
}

}  // namespace

}  // namespace fb
