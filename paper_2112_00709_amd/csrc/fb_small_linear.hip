// The alpha / beta recursions (Eq. 13-14) of small shared graphs that mix, on ordinary numbers in double.
//
// In the log form (fb_small.hip) an arc costs an addition, a maximum, a difference, a conversion and an exponential, and a row
// a logarithm; on probabilities an arc is one multiply-add.  A double reaches from 2^-1022 to 2^1023, so a vector whose
// entries lie within some hundred binary orders of each other - any vector of a graph whose states all reach each other in a
// few steps - is held as probabilities times a power of two, every sum in double.  small_mixes() (fb_small.cpp) picks the
// graphs; left-to-right graphs, where a state that matters may lie any distance behind another, keep the log form.
//
// Work.  NC computing waves walk the arcs from registers as in the log form (the same plan): four gathers, four multiply-adds, one
// product with the frame's factor, one store a row.  L further waves take the frames in turn and do what is not on the chain,
// a row or a frame every L steps each:
//   * the frame's factors 2^(emission - the frame's largest), one per pdf the graph uses, from HBM two rounds ahead, through
//     a polynomial (error 2.6e-9) into one of two rows of LDS;
//   * a finished vector out of LDS, its logarithms (less the largest for float rows), to memory;
//   * the scale.  The wave that has seen the largest entry of vector i puts a power of two into the factors of frame i + L that
//     brings that vector's largest entry to 2^kTarget if nothing else changes it: what the steps between have
//     been scaled by is known (scale_sum), so the lag lets the largest entry stray by what L + 1 steps change it, and nobody on
//     the chain waits for a maximum.
//
// Range.  Weights lie within 2^-100 .. 2^40 and a row's (and column's) sum below 2^40, so the largest entry stays below
// 2^(kTarget + 9 * 40) = 2^860.  A live entry is not below 2^-600 (kLowest), or a factor above zero below 2^-320 (kLowestFactor), without the run
// being given up: a row's sum is then at least 2^-1020, an ordinary double, so nothing above zero is lost unseen.  A run that
// is given up, and one that meets emissions larger than 65536 in size, is done over in the log form by the same workgroup
// (small_again; emissions of that size go straight to its plain form).  The waves that form the factors know of a mask some frames
// ahead: what the first two frames hold ends the run before its first step, what a later one holds some steps behind it (`stop`).
// 701 states over 211 frames, 23 sequences, a direction: 130 us; with a pdf masked by -1e4 in every frame 217 (467 when runs were given up
// behind their last frame only, by functions whose memory accesses all counted as ones to LDS too), in the frame in the middle 285 (467), by
// -1e20 in that frame 549 (913); in the log form at once 253, 253 and 706.  40 states, 100 frames: 28, 50 (70), 67 (70), 157 (195); 43, 43, 169.
//
// What bounds it: with one or two slices a wave the chain of a step (LDS read, three dependent double operations, the lanes of long rows,
// LDS write, barrier: some 400 clocks at 60 states); with 24 slices that chain still: of 1480 clocks a step (2700 in the log form) the LDS is busy for
// 820, 430 of them bank conflicts of its 166 accesses, and a SIMD issues vector instructions in 505 (counted, start and end included).  Figures
// by size stand at small_mixes() in fb_small.cpp.
#include "fb_small_run.h"

namespace fb {

namespace {

constexpr int kTarget = 500, kLowest = -600, kLowestFactor = -320;

template <int NC, int R>
struct LinearShape {
    static constexpr int L = NC <= 4 ? 8 : 4;               // waves beside the computing ones; rows go round them
    static constexpr int NT = (NC + L) * kWave;
    static constexpr int KS = SmallShape<NC, R>::KS, XS = KS + 2;
    static constexpr int U = KS / kWave;                    // states (and pdfs) per lane of such a wave
    static constexpr int kRing = 16;                        // frames whose sums are kept
    // in LDS: two vectors, two before the emission (backward), two rows of factors, the pdfs' bytes in a row of emissions, sums by frame, first maxima, flags
    // The word `stop` takes the first step in which some wave tells that the run leaves the range (as they count up: the least), 1 - kStop
    // if that is known before the first one.
    // Every wave goes by what it read at its last look; a look sees all that has been written in earlier steps (what is written in the
    // same step it may see or not).  Computing waves look when kLook steps begin and decide about the kLook steps behind those: not
    // having seen a word of step n, they go on to step n + 2 kLook - 1 at most.  The others look when a round begins and decide behind it about the
    // next: to step n + 2 L - 1.  So all of them leave the loop in front of the same step, n + kStop.
    static constexpr int kLook = NC <= 2 ? 16 : 8, kStop = 2 * kLook;   // (short steps: a look is 3 % of eight of them)
    static_assert(L <= kLook && kStop >= 2 * kLook && kStop >= 2 * L, "nobody is past the step where all stop");
    static constexpr uint32_t kRow = XS * 8, kPre = 2 * kRow, kFac = 4 * kRow, kFacRow = KS * 8;
    static constexpr uint32_t kPdf = kFac + 2 * kFacRow, kCum = kPdf + KS * 4, kSum = kCum + kRing * 8, kFirst = kSum + kRing * 4, kFlag = kFirst + L * 4, kFin = kFlag + 64;
    static constexpr size_t kBytes = kFin + 8 * NC;
    static_assert(L + 1 < kRing && L <= 8, "sums of the frames under way; flags, and the word `stop` behind them");
};

__device__ unsigned int g_small_restarts;   // diagnostic: runs given up since the library was loaded

// 2^t as m * 2^k: the whole part is k, the rest (-1/2 .. 1/2) goes through the polynomial of degree 6 that meets 2^x at the
// seven Chebyshev nodes there (relative error 2.6e-9; v_exp_f32 has 1e-7).
__device__ __forceinline__ double split_exp2(double t, int &k)
{
    const double w = __builtin_rint(t), f = t - w;
    double m = 0.00015461444691130264;
    m = fma(m, f, 0.0013400428177566465);
    m = fma(m, f, 0.00961805667854805);
    m = fma(m, f, 0.05550327226670292);
    m = fma(m, f, 0.2402265092228862);
    m = fma(m, f, 0.6931472067028327);
    m = fma(m, f, 1.0);
    k = (int)w;
    return m;
}

__device__ __forceinline__ int high_word(double v) { return (int)((uint64_t)__double_as_longlong(v) >> 32); }

// v added up over groups of 2^lg lanes, 1 <= lg <= 6 (short rows first: a branch costs more than the addition)
__device__ __forceinline__ double row_total(double v, int lg, int lane)
{
    v += dpp_mov<0xB1>(v);
    if (lg >= 2) {
        v += dpp_mov<0x4E>(v);
        if (lg >= 3) {
            v += dpp_mov<0x141>(v);
            if (lg >= 4) {
                v += dpp_mov<0x140>(v);
                if (lg >= 5) {
                    const double lo = lane_value(v, 0) + lane_value(v, 16), hi = lane_value(v, 32) + lane_value(v, 48);
                    v = lg == 6 ? lo + hi : (lane < 32 ? lo : hi);
                }
            }
        }
    }
    return v;
}

// the run done over in the log form (plain: in that for large emissions, at once)
template <int NC, int R, int L>
__device__ __attribute__((noinline)) void small_again(__attribute__((address_space(3))) double *lds_raw, uint64_t args, int b_, int which_, int plain_)
{
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    args = (uint64_t)(uint32_t)uniform((int)(uint32_t)args) | (uint64_t)(uint32_t)uniform((int)(uint32_t)(args >> 32)) << 32;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // (rows of the first attempt arrive before these are stored)
    lds_barrier();
    small_run<NC, R, 4, false, L>(*(LaunchParams *)args, args, (double *)lds_raw, uniform(b_), uniform(which_), uniform(plain_) != 0);
}

}  // namespace

// PU: pdfs per lane of a wave of the second kind
template <int NC, int R, int PU>
__global__ __launch_bounds__((LinearShape<NC, R>::NT)) void fb_small_linear_kernel(const RecParams P)
{
    using S = LinearShape<NC, R>;
    constexpr int L = S::L, U = S::U, TM = 4, kDepth = U <= 8 ? 2 : 1;
    extern __shared__ double lds_raw[];
    char *const lds = (char *)lds_raw;
    if (P.started && threadIdx.x == 0) atomicAdd(P.started, 1u);   // this workgroup has its place on a compute unit
    int b, which;
    resolve_sequence<NC>(P, lds_raw, b, which);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const RecDir &D = P.dir[which];
    const bool bwd = D.backward != 0;                       // rows leave before the emission is applied then
    const SmallSub sd = D.small.sub[0];
    const int K = sd.K;
    const int Tn = min(max(P.lengths[b], 0), P.N);
    auto frame = [&](int i) { return bwd ? Tn - 1 - i : i; };
    const size_t out_ld = (size_t)(D.out_ld ? D.out_ld : K), out_at = (size_t)b * P.N * out_ld;
    float *const out_f = (D.out && !D.out_carrier) ? (float *)D.out + out_at : nullptr;
    double *const out_t = (D.out && D.out_carrier) ? (double *)D.out + out_at : nullptr;
    double *const off_seq = D.off ? D.off + (size_t)b * P.N : nullptr;
    double *const cum_ring = (double *)(lds + S::kCum);     // true vector = vector * 2^cum_ring[frame]
    int *const sum_ring = (int *)(lds + S::kSum);           // the scales alone, summed up (scale_sum)
    float *const first_max = (float *)(lds + S::kFirst);
    uint32_t *const flag = (uint32_t *)(lds + S::kFlag);    // [L] the run is to be done over (1), and in the plain form (3)
    volatile __attribute__((address_space(3))) int *const stop = (__attribute__((address_space(3))) int *)(flag + 8);
    double *const fin = (double *)(lds + S::kFin);
    uint32_t again = 0;                                     // (uniform) the flags together
    // the step the loop ends in front of, from what `stop` held
    auto end_of = [&](int word) { return min(Tn, min(__builtin_amdgcn_readfirstlane(word), Tn) + S::kStop); };

    if (Tn > 0 && wave < NC) {
        // ---- computing waves
        uint32_t so[R][TM], tg[R], pl[R];
        double w[R][TM];
        int lg[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int s = wave + j * NC;
            const bool have = s < sd.n_slice;               // (a slice that is not there: every lane adds up nothing)
            const size_t at = (size_t)(sd.slice0 + (have ? s : 0));
            const uint32_t row = have ? D.small.rows[at * kWave + lane] : kSmallNoRow;
            lg[j] = have ? __builtin_amdgcn_readfirstlane(D.small.lg[at]) : 0;
            tg[j] = row == kSmallNoRow ? (uint32_t)S::KS * 8u : row * 8u;
            pl[j] = row == kSmallNoRow ? 0u : (uint32_t)D.small.place[row] * 8u;
#pragma unroll
            for (int t = 0; t < TM; ++t) {
                const Arc a = D.small.arcs[(at * TM + t) * kWave + lane];
                so[j][t] = (uint32_t)a.src;
                w[j][t] = have && a.w > (float)kZeroOut ? exp2((double)a.w) : 0.0;
            }
        }
        lds_barrier();                                      // the first frames' maxima
        lds_barrier();                                      // the factors of frames 0 and 1
#pragma unroll
        for (int j = 0; j < R; ++j) {                       // first frame: start weight (x) emission
            const float s = tg[j] != (uint32_t)S::KS * 8u ? D.bound[tg[j] >> 3] : -INFINITY;
            const double v = s > (float)kZeroOut ? exp2((double)s) : 0.0;
            *(double *)(lds + tg[j]) = v * *(const double *)(lds + S::kFac + pl[j]);
            if (bwd) *(double *)(lds + S::kPre + tg[j]) = v;
        }
        const int first_end = end_of(*stop);
        lds_barrier();
        __builtin_amdgcn_s_setprio(2);                      // (theirs is the chain)
        auto step = [&](auto cc, auto bwd_c) __attribute__((always_inline)) {
            constexpr uint32_t cur = decltype(cc)::value, nxt = cur ^ 1;
            double g[R][TM], fac[R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
#pragma unroll
                for (int t = 0; t < TM; ++t) g[j][t] = *(const double *)(lds + so[j][t] + cur * S::kRow);
                fac[j] = *(const double *)(lds + S::kFac + nxt * S::kFacRow + pl[j]);
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
                double s = fma(g[j][1], w[j][1], g[j][0] * w[j][0]) + fma(g[j][3], w[j][3], g[j][2] * w[j][2]);
                if (lg[j]) s = row_total(s, lg[j], lane);
                if constexpr (decltype(bwd_c)::value) *(double *)(lds + S::kPre + nxt * S::kRow + tg[j]) = s;
                *(double *)(lds + nxt * S::kRow + tg[j]) = s * fac[j];
            }
            lds_barrier();
        };
        auto all_steps = [&](auto bwd_c) __attribute__((always_inline)) {
            int i = 1, end = first_end;
            while (i + 1 < end) {
                int word = *stop;                           // (arrives behind the gathers' backs)
                for (const int last = min(i + S::kLook, end); i + 1 < last; i += 2) {
                    step(std::integral_constant<uint32_t, 0>{}, bwd_c);
                    step(std::integral_constant<uint32_t, 1>{}, bwd_c);
                }
                asm volatile("" : "+v"(word));
                end = end_of(word);
            }
            if (i < end) step(std::integral_constant<uint32_t, 0>{}, bwd_c);
        };
        if (bwd) all_steps(std::true_type{});
        else all_steps(std::false_type{});
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();                                      // the flags
    } else if (Tn > 0) {
        // ---- the other waves
        const int q = wave - NC;
        const int nP = D.small.n_place;
        const bool shifted = !out_t && (out_f || off_seq);  // rows leave without their largest entry
        const float scale = D.out_scale;
        // (lanes behind the last state, or pdf, do the last one again: no lane has to be masked out)
        uint32_t state[U];                                  // the lane's states
        auto place = [&](int l, int u) { return (uint32_t)min(u * kWave + l, nP - 1); };   // (formed where it is used, not kept)
#pragma unroll
        for (int u = 0; u < U; ++u) state[u] = (uint32_t)min(u * kWave + lane, K - 1);
#pragma unroll
        for (int u = 0; u < PU; ++u) {
            *(uint32_t *)(lds + S::kPdf + place(lane, u) * 4) = (uint32_t)D.small.places[place(lane, u)] * 4u;   // (every wave for itself)
        }
        const size_t em_seq = (size_t)b * P.N * P.D;
        auto load = [&](int i, float(&to)[PU]) __attribute__((always_inline)) {
            const char *row = (const char *)(P.emis + em_seq + (size_t)frame(min(i, Tn - 1)) * P.D);
            int l = lane;
            asm volatile("" : "+v"(l));
            uint32_t pdf[PU];
#pragma unroll
            for (int u = 0; u < PU; ++u) pdf[u] = *(const uint32_t *)(lds + S::kPdf + place(l, u) * 4);
#pragma unroll
            for (int u = 0; u < PU; ++u) to[u] = *(const float *)(row + pdf[u]);
        };
        uint32_t size = 0, lowest = ~0u;                    // large emissions; smallest high word above zero, less one
        int lowest_fac = 0;
        auto too_low = [&]() { return (lowest < (uint32_t)((1023 + kLowest) << 20) - 1u) | (lowest_fac < kLowestFactor); };
        auto largest = [&](const float(&e)[PU]) __attribute__((always_inline)) {
            float mx = -INFINITY;
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                mx = tmax(mx, e[u]);
                size = max(size, size_bits(e[u]));
            }
            return lane_value(wave_max_last(mx), kWave - 1);
        };
        auto in_log2 = [](float mx) { return mx > (float)kZero ? (double)mx * kLog2e : 0.0; };   // (a frame nobody can emit: nothing to take off)
        auto factors = [&](int i, const float(&e)[PU], double mx2, int s) __attribute__((always_inline)) {
            char *row = lds + S::kFac + (i & 1) * S::kFacRow;
            int l = lane;
            asm volatile("" : "+v"(l));
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                int k;
                const double m = split_exp2(fma((double)e[u], kLog2e, -mx2), k);
                const bool none = e[u] < (float)kZero;
                k += s;
                lowest_fac = min(lowest_fac, none ? 0 : k);
                *(double *)(row + place(l, u) * 8) = none ? 0.0 : ldexp(m, k);
                if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (four chains at a time: more of them take registers that are not there)
            }
        };
        // emissions asked for ahead: those of the next round, and (kDepth 2) of the one behind it
        float ea[PU], eb[PU], e0[PU];
        load(q, e0);
        load(q + L, ea);
        const float mx0 = largest(e0);
        if (lane == 0) first_max[q] = mx0;
        if (q == 0 && lane == 0) *stop = Tn;
        lds_barrier();
        if (q < 2) factors(q, e0, in_log2(mx0), q == 0 ? kTarget : 0);
        // in step n: what has been seen so far is told
        auto tell = [&](int n) __attribute__((always_inline)) {
            if (__builtin_expect(__any((size > kLargeBits) | too_low()), 0))   // (in assembly: few instructions where it is not so)
                asm volatile("ds_min_i32 %0, %1" :: "v"((uint32_t)(uintptr_t)stop), "v"(n) : "memory");
        };
        tell(1 - S::kStop);                                 // (a label forbidden by a mask, say, is so in every frame: no step at all)
        lds_barrier();
        double cum = -(double)kTarget, cum_before = 0.0;    // of frame q and of the one before it
        for (int j = 0; j <= q; ++j) {
            cum_before = j > 0 ? cum : 0.0;
            cum += in_log2(first_max[j]);
        }
        if (lane == 0) {
            cum_ring[q] = cum;
            sum_ring[q] = kTarget;
        }
        // for rows before the emission everything is one frame back
        double row_cum = bwd ? cum_before : cum;
        int row_sum = bwd && q == 0 ? 0 : kTarget;
        int end = end_of(*stop);
        lds_barrier();                                      // vector 0
        auto bar = [&](int n) { if (n < end) lds_barrier(); };   // the end of step n (kStop is more than L)
        for (int n = 1; n <= q; ++n) {
            if (n + 1 == q) factors(q, e0, in_log2(mx0), 0);
            bar(n);
        }
        if constexpr (kDepth == 2) load(q + 2 * L, eb);
        // All rounds of a wave.  rows: what leaves (0 nothing but the shifts, 1 float rows, 2 double rows); n: states per lane.  Both
        // are constants of the code, so that what is stored behind a round's loads is known and a wait for the loads is not one for the stores.
        double *const off_out = shifted ? off_seq : nullptr;
        float *const cum_out = D.cum ? D.cum + (size_t)b * P.N : nullptr;
        auto rounds = [&](auto rows_c, auto n_c) __attribute__((always_inline)) {
            constexpr int kRows = decltype(rows_c)::value, n = decltype(n_c)::value;
            double v[n];
            int top = 0;                                    // the row's shift, its largest entry: 2^(top + top_l), -1 <= top_l <= 0
            float top_l = 0.0f;
            auto emit = [&](int i, auto part) __attribute__((always_inline)) {   // a third of the lane's entries of row i -> global memory
                constexpr int first = n * decltype(part)::value / 3, last = n * (decltype(part)::value + 1) / 3;
                if constexpr (kRows == 1) {
                    char *orow = (char *)(out_f + (size_t)frame(i) * out_ld);
#pragma unroll
                    for (int u = first; u < last; ++u) {
                        const float l = flog2((float)__builtin_amdgcn_frexp_mant(v[u]));   // (-inf for zero)
                        *(float *)(orow + state[u] * 4) = ((float)(__builtin_amdgcn_frexp_exp(v[u]) - top) + (l - top_l)) * scale;
                    }
                } else if constexpr (kRows == 2) {
                    char *orow = (char *)(out_t + (size_t)frame(i) * out_ld);
#pragma unroll
                    for (int u = first; u < last; ++u) {
                        const float l = flog2((float)__builtin_amdgcn_frexp_mant(v[u]));
                        *(double *)(orow + state[u] * 8) = (row_cum + (double)__builtin_amdgcn_frexp_exp(v[u])) + (double)l;
                    }
                }
            };
            using P0 = std::integral_constant<int, 0>;
            using P1 = std::integral_constant<int, 1>;
            using P2 = std::integral_constant<int, 2>;
            // one round: row i, and the factors of frame i + L from en, which then takes the emissions of a later one.
            // whole: all its L steps and frame i + L are there
            auto round = [&](int i, float(&en)[PU], auto whole) __attribute__((always_inline)) {
                constexpr bool kWhole = decltype(whole)::value;
                // (arithmetic stays in its step: drawn together, two of them make one that the others wait for)
                auto bar = [&](int m) __attribute__((always_inline)) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (kWhole || m < end) lds_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                };
                float hi = 0.0f;                            // (high words of numbers that are not negative, compared as floats)
                int s = 0, sum = 0, high = 0;
                double next_cum = 0.0, mx2 = 0.0;
                auto look = [&]() __attribute__((always_inline)) {
#pragma unroll
                    for (int u = 0; u < n; ++u) {
                        const int h = high_word(v[u]);
                        hi = tmax(hi, __int_as_float(h));
                        lowest = min(lowest, (uint32_t)h - 1u);
                    }
                };
                auto decide = [&]() __attribute__((always_inline)) {
                    int before = 0;
                    if (kWhole) before = sum_ring[(i + L - 1) & (S::kRing - 1)];
                    const int h = lane_value(__float_as_int(wave_max_last(hi)), kWave - 1);
                    top = h ? (h >> 20) - 1022 : 0;
                    high = h;
                    if (kWhole) {
                        sum = __builtin_amdgcn_readfirstlane(before);
                        s = h ? kTarget - top - (sum - row_sum) : 0;
                        if (lane == 0) sum_ring[(i + L) & (S::kRing - 1)] = sum + s;
                    }
                };
                auto shift = [&]() __attribute__((always_inline)) {
                    top_l = high ? flog2((float)__builtin_amdgcn_frexp_mant(__hiloint2double(high, 0))) : 0.0f;
                    if (lane == 0) {
                        const int f = frame(i);
                        if (off_out) off_out[f] = high ? (row_cum + (double)top + (double)top_l) * (double)scale : 0.0;
                        if (kRows != 1 && cum_out) cum_out[f] = 0.0f;   // (carrier rows are not shifted)
                    }
                };
                auto centre = [&]() __attribute__((always_inline)) {
                    if constexpr (kWhole) {
                        const double before = cum_ring[(i + L - 1) & (S::kRing - 1)];
                        mx2 = in_log2(largest(en));
                        const double after = before + (mx2 - (double)s);
                        if (lane == 0) cum_ring[(i + L) & (S::kRing - 1)] = after;
                        next_cum = bwd ? before : after;
                    }
                };
                auto prepare = [&]() __attribute__((always_inline)) {
                    if constexpr (kWhole) factors(i + L, en, mx2, s);
                };
                auto request = [&]() __attribute__((always_inline)) {
                    if constexpr (kWhole) load(i + (1 + kDepth) * L, en);
                };
                const char *row = lds + (bwd ? S::kPre : 0u) + (i & 1) * S::kRow;
#pragma unroll
                for (int u = 0; u < n; ++u) v[u] = *(const double *)(row + state[u] * 8);
                int word = 0;
                if (kWhole) {
                    word = *stop;                           // (the look of this round: for the next one)
                    // (in step i + 1, of the round before: behind the factors it would be in the longest of a round's steps, which all
                    // waves wait for: 16 states 28 -> 36 us, 701 states 137 -> 152)
                    tell(i + 1);
                }
                if constexpr (L == 4) {
                    look();
                    bar(i + 1);
                    decide();
                    shift();
                    emit(i, P0{});
                    bar(i + 2);
                    centre();
                    prepare();
                    bar(i + 3);
                    request();
                    emit(i, P1{});
                    emit(i, P2{});
                    bar(i + 4);
                } else {
                    bar(i + 1);
                    look();
                    decide();
                    bar(i + 2);
                    shift();
                    emit(i, P0{});
                    bar(i + 3);
                    emit(i, P1{});
                    bar(i + 4);
                    emit(i, P2{});
                    bar(i + 5);
                    centre();
                    bar(i + 6);
                    prepare();
                    bar(i + 7);
                    request();
                    bar(i + 8);
                }
                row_cum = next_cum;
                row_sum = bwd ? sum : sum + s;
                if (kWhole) end = end_of(word);
            };
            int i = q;
            // (two copies of a round, not a third for an odd last one: a short sequence meets each for the first time, and waits for the code)
            for (; i + L < end; i += L) {
                round(i, ea, std::true_type{});
                if constexpr (kDepth == 2) {
                    i += L;
                    if (i + L >= end) break;
                    round(i, eb, std::true_type{});
                }
            }
            if (i < end) round(i, ea, std::false_type{});   // (no emissions are asked of a last round)
        };
        auto sized = [&](auto rows_c) __attribute__((always_inline)) {
            if constexpr (U == 16) {
                if (K <= 8 * kWave) { rounds(rows_c, std::integral_constant<int, 8>{}); return; }
                if (K <= 12 * kWave) { rounds(rows_c, std::integral_constant<int, 12>{}); return; }
            }
            rounds(rows_c, std::integral_constant<int, U>{});
        };
        if (out_f) sized(std::integral_constant<int, 1>{});
        else if (out_t) sized(std::integral_constant<int, 2>{});
        else sized(std::integral_constant<int, 0>{});
        const uint32_t f = __any(size > kLargeBits) ? 3u : __any(too_low()) ? 1u : 0u;
        if (lane == 0) flag[q] = f;
        lds_barrier();
    }
    if (Tn > 0) {
        for (int i = 0; i < L; ++i) again |= flag[i];
        again = (uint32_t)__builtin_amdgcn_readfirstlane((int)again);
    }
    if (__builtin_expect(again != 0, 0)) {
        if (threadIdx.x == 0) atomicAdd(&g_small_restarts, 1u);
        small_again<NC, R, L>((__attribute__((address_space(3))) double *)lds_raw, (uint64_t)__builtin_amdgcn_kernarg_segment_ptr(), b, which, again >> 1);
    } else {
        if (Tn > 0) {
            // ---- log Z from the last vector and the end weights, by the computing waves
            if (wave < NC) {
                const double *xl = (const double *)(lds + ((Tn - 1) & 1) * S::kRow);
                double z = 0.0;
                for (int k = wave * kWave + lane; k < K; k += NC * kWave) {
                    const float o = D.obound[k];
                    z += o > (float)kZeroOut ? xl[k] * exp2((double)o) : o != o ? (double)o : 0.0;
                }
                z = group_all(z, 6, lane, [](double x, double y) { return x + y; });
                if (lane == 0) fin[wave] = z;
            }
            __syncthreads();
            if (threadIdx.x == 0 && D.logz) {
                double z = fin[0];
                for (int v = 1; v < NC; ++v) z += fin[v];
                D.logz[b] = z == 0.0 ? -INFINITY : (log2(z) + cum_ring[(Tn - 1) & (S::kRing - 1)]) * kLn2;
            }
        } else if (threadIdx.x == 0 && D.logz) {
            D.logz[b] = -INFINITY;
        }
        small_pad<S::NT>(D.fill_pad != 0, out_f, off_seq, out_ld, Tn, P.N, K);
    }
    count_done(P);
}

template <int NC, int R, int PU>
static int launch_pdfs(const RecParams &p, void *stream)
{
    using S = LinearShape<NC, R>;
    constexpr size_t lds = std::max(S::kBytes, SmallShape<NC, R, S::L>::lds_bytes(true, false));
    static_assert(lds <= 64 * 1024, "on-chip memory of a launch without a raised limit");
    const int32_t n_seq = p.order ? p.n_launch : p.B;
    hipLaunchKernelGGL((fb_small_linear_kernel<NC, R, PU>), dim3((unsigned)(n_seq * p.n_dir)), dim3(S::NT), lds, (hipStream_t)stream, p);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? FB_OK : fail(FB_EHIP, std::string("small-graph kernel launch: ") + hipGetErrorString(e));
}

template <int NC, int R>
static int launch_variant(const RecParams &p, void *stream)
{
    constexpr int U = LinearShape<NC, R>::U;
    const int n = p.dir[0].small.n_place;
    if (U > 4 && n <= 2 * kWave) return launch_pdfs<NC, R, (U > 4 ? 2 : U)>(p, stream);
    if (U > 8 && n <= 5 * kWave) return launch_pdfs<NC, R, (U > 8 ? 5 : U)>(p, stream);
    return launch_pdfs<NC, R, U>(p, stream);
}

unsigned int small_linear_restarts()
{
    unsigned int n = 0;
    return hipMemcpyFromSymbol(&n, HIP_SYMBOL(g_small_restarts), sizeof(n)) == hipSuccess ? n : 0u;
}

// A workgroup with one computing wave (up to two slices) has eight others here, and a wave up to 168 registers: one such workgroup fits a
// compute unit, where four of the log form's three waves do.  More workgroups than compute units of so small a graph therefore run in that form.  A
// direction, us, here / in the log form: 16 states, 50 frames, 256 sequences 15 / 21, 512 27 / 23, 1024 52 / 24; over 200 frames 38 / 65, 73 / 72, 143 / 75;
// 60 states, 50 frames 19 / 26, 36 / 29, 69 / 32.  Of more computing waves the log form too fits once: 120 states, 1024 sequences, 50 frames 89 / 109.
bool small_linear_pays(int slices, int64_t workgroups)
{
    static const int n_cu = [] {
        int dev = 0, n = 0;
        return hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0 ? n : 256;
    }();
    return slices > 2 || workgroups <= n_cu;
}

int launch_small_linear(const RecParams &p, int slices, void *stream)
{
    for (int i = 0; i < p.n_dir; ++i)
        if (!p.dir[i].small.places || !p.shared || p.dir[i].small.n_place < 1) return fail(FB_EHIP, "internal error: small-graph launch without its list of pdfs");
    if (p.Kcap > kSmallStates) return fail(FB_EHIP, "internal error: small-graph launch");
    if (slices <= 1) return launch_variant<1, 1>(p, stream);
    if (slices <= 2) return launch_variant<1, 2>(p, stream);
    if (slices <= 4) return launch_variant<2, 2>(p, stream);
    if (slices <= 8) return launch_variant<4, 2>(p, stream);
    if (slices <= 16) return launch_variant<8, 2>(p, stream);
    if (slices <= 24) return launch_variant<8, 3>(p, stream);
    if (slices <= kSmallMaxSlices) return launch_variant<8, 4>(p, stream);
    return fail(FB_EHIP, "internal error: small-graph launch");
}

}  // namespace fb
