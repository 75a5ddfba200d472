// gfx950 kernels of libfb_amd: the alpha / beta recursions (Eq. 13-14), the
// posteriors (Eq. 15) with their accumulation over tied states, and the LF-MMI
// objective (Eq. 16).
//
// Work decomposition.  Sequences of a batch are independent (the batched
// transition matrix is block diagonal), while the frames of one sequence are
// strictly sequential.  One workgroup therefore owns one (sequence, direction)
// pair for the whole time loop and keeps that sequence's state vector in LDS:
// a time step needs workgroup barriers only, never a grid-wide one, and the
// forward and backward recursions of a batch run side by side in one launch.
// Within a step the sparse product is walked one matrix row per lane along a
// static row-split sliced-ELL schedule (fb_sell.cpp) flattened into one stream of
// arcs per wave (fb_stream.cpp) that is prefetched several batches ahead; the arcs
// come from L2, the gathered vector from LDS.
//
// Arithmetic.  Internally logs are base 2 (weights and emissions are scaled by
// log2 e once), so the semiring sum is v_exp_f32 / v_log_f32 with no
// multiplications.  A row's (+)-sum is evaluated in one pass with a running
// maximum: one exponential per arc, one logarithm per row.  The state vector is
// kept normalised: every step subtracts the previous step's maximum, the
// subtracted amounts are the offsets handed back to the caller and their sum is
// accumulated in double for log Z.  The vector's element type ("carrier") is
// float or double; exponentials and logarithms are single precision either way
// (they act on differences to the running maximum, which are small).  One
// instantiation (LINW) takes the arc weights as 2^w and multiplies: see
// stream_linear_weights for when a graph gets it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "fb_device.h"
#include "fb_internal.h"

namespace fb {

// ---------------------------------------------------------------------------
// alpha / beta recursion.  grid = B * n_dir workgroups of NW waves; workgroup
// (b, which) runs direction dir[which] of sequence b over all its frames.
//
// With x_n the vector kept in LDS, both directions are the same recursion on a
// matrix and its transpose:
//   forward   x_n = alpha_n              = v_n o (+)_{in(j)}  (w (x) x_{n-1}[src])
//   backward  x_n = beta_n (x) v_n       = v_n o (+)_{out(i)} (w (x) x_{n+1}[dst])
// and beta_n itself is the row sum before v_n is applied.
//
// Waves 0..NW-2 compute: their only global-memory traffic inside the time loop
// is their own arc stream, a fixed sequence of loads that stays ahead of its
// use across barriers and across time steps; the LDS gathers of a batch are
// issued one batch ahead of the arithmetic that consumes them.  Wave NW-1 moves
// data: it brings the next frame's emissions from HBM straight into LDS, copies
// the finished vector of the previous step out, keeps the offsets and log Z.
// HBM latency therefore never sits in front of an arc load.
//
// LDS of a workgroup (carrier type T unless noted):
//   xb   2 x Xs   x of the previous / current step; Xs = Kcap + Ccap + 1: the
//                 states, then the clones of rows too long for one slice, then a dump slot
//   bh   2 x Xs   beta before v is applied (backward direction only)
//   red  4 x NW   step maxima, scratch of the last reduction.  Float vectors: the maximum of step i is
//                 word i % 3, reached by one LDS atomic maximum per wave; the data-moving wave clears
//                 the word of the step after next.  Double vectors: one slot per wave and parity.
//   er   3 x (Ecap + 1) float   emissions as given (natural log) of the frame in use and
//                               of the next two; slot Ecap = 0
//   pix  Ecap int32             packed graphs: pdf id of every state
//   vix  Xs uint16              which staged emission every target (state, clone, dump slot) takes
//   bpb  2 x Xs uint16          tropical semiring only: back-pointers of the previous / current step
//
// XF != 0: the state buffers have the fixed length XF (>= Kcap + Ccap + 1) whatever the graph.  The
// time loop is then unrolled over the two buffer parities, every buffer address is a compile-time
// constant, and a gather is one ds_read whose address register is the arc's source field as stored
// (a byte offset) with the buffer in the instruction's offset field.
// ---------------------------------------------------------------------------
// One (sequence, direction) pair from its first frame to its last, by the whole workgroup.
template <int NW, class T, bool TROP, int XF, bool LINW = false>
__device__ __forceinline__ void recursion_run(const RecParams &P, const int b, const int which, double *lds_raw)
{
    static_assert(!LINW || (!TROP && XF != 0), "weights as 2^w: log semifield, fixed buffers");
    constexpr int NRES = kResident;
    constexpr int NT = NW * kWave, NC = NW - 1;
    const T kNegInf = (T)(-INFINITY);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool io_wave = wave == NC;
    const RecDir &R = P.dir[which];
    const StreamDev &S = R.sched;
    const bool bwd = R.backward != 0, keep_pre = bwd && !TROP;   // keep_pre: rows leave before the emission is applied
    const SubDesc sd = S.sub[P.shared ? 0 : b];
    const int K = sd.K, k0 = sd.k0, nC = sd.n_slot;
    const int Tn = min(max(P.lengths[b], 0), P.N);
    const int mid = path_middle(Tn);
    const int Ts = Tn > 0 && TROP ? (bwd ? Tn - mid : mid + 1) : Tn;   // frames this direction visits
    const int nE = P.shared ? P.D : K;           // entries of a staged emission vector
    const int nX = P.Kcap + R.Ccap + 1;          // states, clone slots, dump slot
    const int Xs = XF ? XF : nX, Es = P.Ecap + 1;

    T *xb = (T *)lds_raw;
    T *bh = xb + 2 * Xs;
    T *red = bh + (keep_pre ? 2 * Xs : 0);
    float *er = (float *)(red + 4 * NW + 2);
    int32_t *pix = (int32_t *)(er + 3 * Es);
    uint16_t *vix = (uint16_t *)(pix + (P.shared ? 0 : P.Ecap));   // emission index of every target
    uint16_t *bpb = vix + ((Xs + 1) & ~1);                         // tropical semiring: 2 x Xs back-pointers
    constexpr int kSrcShift = sizeof(T) == 4 ? 2 : 3;              // an arc's source field is index << kSrcShift

    const float *em_seq = P.emis + (size_t)b * P.N * P.D;
    const size_t out_ld = P.shared ? (size_t)(R.out_ld ? R.out_ld : K) : (size_t)P.Ktot;
    const size_t out_at = P.shared ? (size_t)b * P.N * out_ld : (size_t)k0;
    float *out_f = (R.out && !R.out_carrier) ? (float *)R.out + out_at : nullptr;
    T *out_t = (R.out && R.out_carrier) ? (T *)R.out + out_at : nullptr;
    double *off_seq = R.off ? R.off + (size_t)b * P.N : nullptr;
    auto frame = [&](int i) { return bwd ? Tn - 1 - i : i; };
    // the maximum over the workgroup of the vector of step i (the next step normalises by it)
    constexpr bool kAtomMax = sizeof(T) == 4;
    auto put_max = [&](int i, T wmax) {
        // (a double carrier's maximum is reduced as a float rounded up: what the next step subtracts from every entry
        // need only be near the largest, the same for all, and not below it by more than rounding)
        float wm;
        if constexpr (sizeof(T) == 8) wm = wave_max_last(__double2float_ru((double)wmax));
        else wm = wave_max_last(wmax);
        if (lane == kWave - 1) {   // (one lane per wave: atomics of many lanes on one word are served one at a time)
            if constexpr (kAtomMax) lds_raise((float *)red + i % 3, wm);
            else red[(i & 1) * NW + wave] = (T)wm;
        }
    };
    auto get_max = [&](int i) {
        if constexpr (kAtomMax) {
            return red[i % 3];
        } else {
            T M = red[(i & 1) * NW];
#pragma unroll
            for (int w = 1; w < NW; ++w) M = tmax(M, red[(i & 1) * NW + w]);
            return M;
        }
    };

    // ---- duties of the data-moving wave (called by that wave only, all 64 lanes)
    // Packed graphs: the pdf of the lane's states u * 64 + lane, in registers when a (sub-)graph has at most
    // kPixRegs * 64 states (read once: looked up in LDS at every frame, each of a frame's loads would wait for a read)
    // (the small-graph instantiations only: the others have no registers to spare)
    constexpr int kPixRegs = NW == kNWSmall ? 8 : 0;
    const bool pix_in_regs = kPixRegs > 0 && !P.shared && nE <= kPixRegs * kWave;
    int32_t pixr[kPixRegs > 0 ? kPixRegs : 1] = {};
    // emissions of frame f -> dst, through the direct global->LDS path (no registers, any length)
    auto stage = [&](int f, float *dst) {
        const float *row = em_seq + (size_t)f * P.D;
        if (P.shared) {
            if ((P.D & 3) == 0 && ((uintptr_t)row & 15) == 0) {
                for (int e0 = 0; e0 < nE; e0 += 4 * kWave)
                    if (e0 + 4 * lane < nE)
                        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + e0 + 4 * lane),
                                                         (__attribute__((address_space(3))) void *)(dst + e0), 16, 0, 0);
            } else {
                for (int e0 = 0; e0 < nE; e0 += kWave)
                    if (e0 + lane < nE)
                        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + e0 + lane),
                                                         (__attribute__((address_space(3))) void *)(dst + e0), 4, 0, 0);
            }
        } else if (kPixRegs > 0 && pix_in_regs) {
#pragma unroll
            for (int u = 0; u < kPixRegs; ++u)
                if (u * kWave < nE && u * kWave + lane < nE)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + pixr[u]),
                                                     (__attribute__((address_space(3))) void *)(dst + u * kWave), 4, 0, 0);
        } else {
            for (int e0 = 0; e0 < nE; e0 += kWave)
                if (e0 + lane < nE)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + pix[e0 + lane]),
                                                     (__attribute__((address_space(3))) void *)(dst + e0), 4, 0, 0);
        }
    };
    auto staged_wait = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    // a finished vector -> global memory, coalesced; a cloned state leaves as the (+)-sum of its clones
    const CloneDesc *cdesc = S.clones + sd.clone0;
    // (copies go in groups of several pieces per lane, all read before any is stored: a store's data registers
    // can only be reused once the store has completed, so a read-one-store-one loop would pay a full HBM
    // round trip per piece)
    auto copy_out = [&](auto *orow, const auto *srcv, int n, auto cvt) {
        constexpr int U = NW == kNWShared ? 16 : 8;   // (small graphs: a row of up to 512 states is one group)
        for (int k0 = 0; k0 < n; k0 += U * kWave) {
            std::remove_cv_t<std::remove_reference_t<decltype(srcv[0])>> v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = srcv[min(k0 + u * kWave + lane, n - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u) asm volatile("" : "+v"(v[u]));   // every read stays in front of the stores
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + u * kWave + lane < n) orow[k0 + u * kWave + lane] = cvt(v[u]);
        }
    };
    auto write_row = [&](int f, const T *srcv) {
        if (out_f) {
            float *orow = out_f + (size_t)f * out_ld;
            const float scale = R.out_scale;
            copy_out(orow, srcv, K, [scale](T x) { return (float)x * scale; });
        } else if (out_t) {
            T *orow = out_t + (size_t)f * out_ld;
            if (sizeof(T) == 4 && (out_ld & 3) == 0 && (size_t)((K + 3) & ~3) <= out_ld && ((uintptr_t)orow & 15) == 0 &&
                ((uintptr_t)srcv & 15) == 0) {
                // whole 16-byte pieces; when K is not a multiple of 4 the last one takes up to 3 values that lie
                // behind the states in LDS into the row's padding, which nobody reads
                const float4 *s4 = (const float4 *)srcv;
                float4 *o4 = (float4 *)orow;
                constexpr int U = 8;
                const int n4 = (K + 3) / 4;
                for (int k0 = 0; k0 < n4; k0 += U * kWave) {
                    float4 v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = s4[min(k0 + u * kWave + lane, n4 - 1)];
#pragma unroll
                    for (int u = 0; u < U; ++u)   // every read stays in front of the stores
                        asm volatile("" : "+v"(v[u].x), "+v"(v[u].y), "+v"(v[u].z), "+v"(v[u].w));
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (k0 + u * kWave + lane < n4) o4[k0 + u * kWave + lane] = v[u];
                }
            } else {
                copy_out(orow, srcv, K, [](T x) { return x; });
            }
        }
        if (out_f || out_t)
            for (int j = lane; j < sd.n_cdesc; j += kWave) {   // stores of one wave to one address keep their order
                const CloneDesc cd = cdesc[j];
                T m = (T)kNegBig;
                float s = 0.0f;
                lse_add(m, s, srcv[cd.state]);
                for (int i = 0; i < cd.count; ++i) lse_add(m, s, srcv[P.Kcap + cd.first + i]);
                const T v = m + (T)flog2(s);
                if (out_f) out_f[(size_t)f * out_ld + cd.state] = (float)v * R.out_scale;
                else out_t[(size_t)f * out_ld + cd.state] = v;
            }
    };

    // tropical semiring: the back-pointers of step i (i >= 1) -> global memory; a row holds the states
    // and, behind them, the clone slots (a back-pointer is an index into the state buffer: a state, or
    // Kcap + slot for a clone)
    auto write_bp = [&](int i, const uint16_t *srcb) {
        if (TROP && R.bp) {
            const int f = bwd ? Tn - i : i;   // (row f joins frames f - 1 and f, see path_middle)
            uint16_t *orow = R.bp + (P.shared ? ((size_t)b * P.N + f) * R.bp_ld : (size_t)f * R.bp_ld);
            uint16_t *ost = orow + (P.shared ? 0 : k0), *ocl = orow + (P.shared ? K : P.Ktot + b * R.bp_ccap);
            copy_out(ost, srcb, K, [](uint16_t x) { return x; });
            copy_out(ocl, srcb + P.Kcap, nC, [](uint16_t x) { return x; });
        }
    };

    if (Tn > 0) {
        // ---- first frame of this direction: x = start weight (x) v
        if (!P.shared)
            for (int k = tid; k < K; k += NT) pix[k] = P.pdf[k0 + k];
        for (int k = tid; k < nX; k += NT) vix[k] = S.vix[(size_t)(P.shared ? 0 : b) * nX + k];
        if (tid < 3) er[tid * Es + P.Ecap] = 0.0f;   // the emission of rows that take none
        if (kAtomMax && tid < 3) red[tid] = kNegInf;
        __syncthreads();
        if (io_wave) {
            if (kPixRegs > 0 && pix_in_regs) {
#pragma unroll
                for (int u = 0; u < kPixRegs; ++u) pixr[u] = u * kWave + lane < nE ? pix[u * kWave + lane] : 0;
            }
            stage(frame(0), er);
            if (Ts > 1) stage(frame(1), er + Es);
            staged_wait();
            if (Ts > 2) stage(frame(2), er + 2 * Es);   // lands while step 1 runs
            if (off_seq && lane == 0) off_seq[frame(0)] = 0.0;
            if (R.cum && lane == 0) R.cum[(size_t)b * P.N + frame(0)] = 0.0f;
        }
        __syncthreads();
        T wmax = kNegInf;
        for (int k = tid; k < K; k += NT) {
            const T s = (T)R.bound[k0 + k];
            // (a best path's backward recursion ends before the emission of its last frame, which may be this one)
            const T x = TROP && bwd && Ts == 1 ? s : s + (T)er[P.shared ? P.pdf[k0 + k] : k] * (T)kLog2e;
            xb[k] = x;
            if (keep_pre) bh[k] = s;
            wmax = tmax(wmax, x);
        }
        for (int k = tid; k < nC; k += NT) {   // clones start empty: the state itself holds the start weight
            xb[P.Kcap + k] = kNegInf;
            if (keep_pre) bh[P.Kcap + k] = kNegInf;
        }
        if (tid == 0) xb[nX - 1] = xb[Xs + nX - 1] = kNegInf;   // the dump slot holds zero-bar in both buffers, always
        put_max(0, wmax);
        lds_barrier();

        double csum = 0.0;
        if (io_wave) {
            for (int i = 1; i < Ts; ++i) {
                const int cur = (i - 1) & 1;
                const T M = get_max(i - 1);
                const T c = (M == kNegInf) ? (T)0 : M;
                csum += (double)c;
                if (off_seq && lane == 0) off_seq[frame(i)] = csum * (double)R.out_scale;
                if (R.cum && lane == 0) R.cum[(size_t)b * P.N + frame(i)] = (float)csum;
                staged_wait();   // frame i+1, requested a whole step ago, is in LDS
                if (i + 2 < Ts) stage(frame(i + 2), er + ((i + 2) % 3) * Es);   // buffer of frame i-1: no longer read
                write_row(frame(i - 1), keep_pre ? bh + cur * Xs : xb + cur * Xs);
                if (TROP && i >= 2) write_bp(i - 1, bpb + cur * Xs);
                if (lane == 0) {   // its own slot counts for nothing / the word of step i + 1 starts empty
                    if (kAtomMax) red[(i + 1) % 3] = kNegInf;
                    else red[(i & 1) * NW + wave] = kNegInf;
                }
                __syncthreads();
            }
        } else {
            const WaveDesc wd = S.waves[sd.wave_ptr0 + wave];
            // a lane's share of a batch is two 16-byte pieces: rows 0-1 and rows 2-3
            // (the address is a wave-uniform base plus the lane's 16 bytes: no per-lane 64-bit arithmetic)
            const uint64_t arc_base = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)wd.arc_base) |
                                      ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(wd.arc_base >> 32)) << 32);
            const float4 *stream = (const float4 *)(S.arcs + arc_base);
            auto load_from = [&](Arc(&dst)[kBatchRows], const float4 *p) {   // p: the lane's first piece
                const float4 lo = p[0], hi = p[kWave];
                dst[0] = Arc{(int32_t)__float_as_uint(lo.x), lo.y};
                dst[1] = Arc{(int32_t)__float_as_uint(lo.z), lo.w};
                dst[2] = Arc{(int32_t)__float_as_uint(hi.x), hi.y};
                dst[3] = Arc{(int32_t)__float_as_uint(hi.z), hi.w};
            };
            // The first NRES batches of the wave's step stay in registers for the whole time loop;
            // the rest of the stream is re-read every step through a ring that runs kRing-1 batches
            // ahead of its use, across barriers and across steps (it holds graph data only).
            Arc res[NRES][kBatchRows];
#pragma unroll
            for (int q = 0; q < NRES; ++q) load_from(res[q], stream + (size_t)q * (2 * kWave) + lane);
            // streamed part: rp0 = the lane's piece of its first batch, rp = of the batch to request next (the
            // requests walk the part cyclically, so the pointer moves by one batch per request and goes back
            // to rp0 once per time step, at a place every step knows: no index arithmetic per batch)
            const float4 *const rp0 = stream + (size_t)NRES * (2 * kWave) + lane;
            const float4 *rp = rp0;
            const int n_iter = wd.n_iter;
            // flag bytes: words 0-1 of the wave hold those of the resident batches, then one word per
            // iteration; kept in registers (word i in lane i) and read with v_readlane
            const uint32_t *fwp = S.flagwords + wd.flag_base;
            const uint32_t rflag0 = fwp[0], rflag1 = fwp[1];
            // batches of the resident part that hold arcs (padding only follows them, and only when nothing is streamed)
            int n_res = 0;
            for (int q = 0; q < NRES; ++q)
                if (!((((q < 4 ? rflag0 : rflag1) >> (8 * (q & 3))) & 0xffu) & kFlagSkip)) n_res = q + 1;
            n_res = __builtin_amdgcn_readfirstlane(n_res);
            const uint32_t fwv0 = lane < n_iter ? fwp[2 + lane] : 0u;
            const uint32_t fwv1 = lane + kWave < n_iter ? fwp[2 + lane + kWave] : 0u;
            Arc ring[kRing][kBatchRows];
            if (n_iter > 0) {
#pragma unroll
                for (int j = 0; j + 1 < kRing; ++j) {
                    load_from(ring[j], rp);
                    rp += 2 * kWave;
                    __builtin_amdgcn_sched_barrier(0);   // keep the issue order: waits count loads in order
                }
            }
            // gathered values of the batch being folded and of the next one; the buffers rotate with the batch
            // number, and an unrolled iteration must bring the rotation back to where it started
            constexpr int GB = kRing % 2 == 0 ? 2 : 3;
            static_assert(kRing % GB == 0, "ring size must be a multiple of the gather buffer count");
            T g[GB][kBatchRows];
            // Source fields are byte offsets into the buffer vbase.  With fixed buffers the workgroup's LDS
            // starts at address 0 (the host launches this instantiation only if the kernel has no static LDS)
            // and the buffer sits at a constant address, so the load takes the field itself as its address.
            // The source field of a batch's last row carries the row's target in its upper half when the batch
            // closes a slice (zero otherwise: offsets stay below 64 KB), so its lower half is the source either way.
            // stacked: the batch holds the rows of several stacked slices, whose parts all end with a target in
            // the upper half (only the first kMaxStacked batches of a step can be: the flag is a constant false elsewhere)
            auto gather = [&](T(&dst)[kBatchRows], const Arc(&a)[kBatchRows], const T *vbase, bool stacked) {
                auto at = [&](int32_t off) {
                    if constexpr (XF != 0) {
                        typedef const __attribute__((address_space(3))) T lds_ct;
                        const uint32_t addr = (uint32_t)off + (vbase == xb ? 0u : (uint32_t)(XF * sizeof(T)));
                        return *(lds_ct *)(uintptr_t)addr;
                    } else {
                        return *(const T *)((const char *)vbase + off);
                    }
                };
                if (stacked) {
#pragma unroll
                    for (int r = 0; r < kBatchRows; ++r) {
                        uint32_t s = (uint32_t)a[r].src;
                        asm volatile("" : "+v"(s));   // (not hoisted out of the time loop: see target() below)
                        dst[r] = at((int32_t)(s & 0xffffu));
                    }
                } else {
#pragma unroll
                    for (int r = 0; r + 1 < kBatchRows; ++r) dst[r] = at(a[r].src);
                    dst[kBatchRows - 1] = at((int32_t)((uint32_t)a[kBatchRows - 1].src & 0xffffu));
                }
            };

            // one time step; curc: parity of the buffer that holds the previous step (an int, or a
            // compile-time constant when the buffers have fixed addresses)
            auto step = [&](int i, auto curc) {
                const int cur = curc, nxt = cur ^ 1;
                const T *xc = xb + cur * Xs;
                T *xn = xb + nxt * Xs;
                T *bn = bh + nxt * Xs;
                const float *ern = er + (i % 3) * Es;
                // Waves of equal priority are served oldest first, so with one fixed priority the younger waves of
                // a SIMD would do most of their step alone after the older ones have finished theirs.  A wave's
                // priority therefore falls as its step advances: whoever has more left goes first, and the waves
                // of a SIMD reach the barrier together.  The younger half of the waves stays one level above the
                // older half, which would otherwise still win every tie.
                const bool young = wave >= NW / 2;
                auto prio = [&](auto level) {   // level: a compile-time constant 1..3
                    if (NW == kNWShared) {
                        if (young) __builtin_amdgcn_s_setprio(decltype(level)::value);
                        else __builtin_amdgcn_s_setprio(decltype(level)::value - 1);
                    }
                };
                prio(std::integral_constant<int, 3>{});
                const T M = get_max(i - 1);
                const T c = (M == kNegInf) ? (T)0 : M;
                wmax = kNegInf;
                const bool no_em = TROP && bwd && i == Ts - 1;   // (see the first frame)
                auto emitted = [&](float e) { return TROP && no_em ? (T)0 : (T)e * (T)kLog2e; };
                T m = TROP ? kNegInf : (T)kNegBig;
                float sum = 0.0f;
                int arg = 0;                         // tropical semiring: the state the best term so far came from
                uint16_t *bpn = bpb + nxt * Xs;
                const T *vbase = xc;
                if (i <= 2)   // rows without arcs: the semiring zero from the second frame on, in both buffers
                    for (int z = tid; z < sd.n_zero; z += NC * kWave) {
                        const int k = S.zero_rows[sd.zero0 + z];
                        xn[k] = kNegInf;
                        if (keep_pre) bn[k] = kNegInf;
                    }
                // fold one batch: a, gv = its entries and gathered values; next = the batch after it (its
                // gathers are issued before this batch's arithmetic), has_next: there is one
                // res: the batch is one of the first kMaxStacked of the step (the only ones that may be stacked);
                // next_stacked: the batch after it is a stacked one
                auto fold = [&](auto res, uint32_t f, const Arc(&a)[kBatchRows], const T(&gv)[kBatchRows], T(&gnext)[kBatchRows],
                                const Arc(&next)[kBatchRows], bool next_stacked, bool has_next) {
                    if (has_next) gather(gnext, next, vbase, next_stacked);
                    if (decltype(res)::value && (f & (kFlagDual | kFlagQuad))) {
                        // Stacked slices: every part of the lane is a row of its own with one or two terms, closed
                        // here; the running sums of the lane are not touched (stacked batches come first).
                        // val: the part's (+)-sum; parg: tropical semiring, where its best term came from
                        // The emissions of the parts' targets first, all of them (two LDS reads in a row each, one
                        // after the other per part they would be most of a small graph's time step).
                        const bool quad = (f & kFlagQuad) != 0;
                        uint32_t ptgt[kBatchRows];
                        float pem[kBatchRows];
#pragma unroll
                        for (int r = 0; r < kBatchRows; ++r) {
                            uint32_t field = (uint32_t)a[(quad || (r & 1)) ? r : r + 1].src;   // two parts: rows 1 and 3 name the targets
                            asm volatile("" : "+v"(field));
                            ptgt[r] = field >> 16;
                        }
                        uint32_t pvi[kBatchRows];
#pragma unroll
                        for (int r = 0; r < kBatchRows; ++r) pvi[r] = vix[ptgt[r]];
#pragma unroll
                        for (int r = 0; r < kBatchRows; ++r) pem[r] = ern[pvi[r]];
                        auto close_part = [&](T val, int parg, int r) {   // r: a row of the part that names its target
                            const uint32_t tgt = ptgt[r];
                            const T pre = val - c;
                            const T x = pre + emitted(pem[r]);
                            xn[tgt] = x;
                            if constexpr (TROP) bpn[tgt] = (uint16_t)(parg >> kSrcShift);
                            else if (keep_pre) bn[tgt] = pre;
                            wmax = tmax(wmax, x);
                        };
                        T xs[kBatchRows];
#pragma unroll
                        for (int r = 0; r < kBatchRows; ++r) xs[r] = gv[r] + (T)a[r].w;
                        if (f & kFlagQuad) {
#pragma unroll
                            for (int r = 0; r < kBatchRows; ++r) {   // one term: the sum is the term
                                const uint32_t field = (uint32_t)a[r].src;
                                if constexpr (TROP) close_part(xs[r], xs[r] > kNegInf ? (int)(field & 0xffffu) : 0, r);
                                else close_part(xs[r] > (T)kNegBig ? xs[r] : kNegInf, 0, r);   // (as the running sums treat it)
                            }
                        } else {
#pragma unroll
                            for (int p = 0; p < 2; ++p) {
                                const T u0 = xs[2 * p], u1 = xs[2 * p + 1];
                                const uint32_t field = (uint32_t)a[2 * p + 1].src;
                                if constexpr (TROP) {
                                    T pm = kNegInf;
                                    int parg = 0;
                                    if (u0 > pm) { pm = u0; parg = a[2 * p].src; }
                                    if (u1 > pm) { pm = u1; parg = (int)(field & 0xffffu); }
                                    close_part(pm, parg, 2 * p + 1);
                                } else {
                                    const T pm = tmax3((T)kNegBig, u0, u1);
                                    close_part(pm + (T)flog2(fexp2((float)(u0 - pm)) + fexp2((float)(u1 - pm))), 0, 2 * p + 1);   // 0 -> -inf
                                }
                            }
                        }
                    } else if (!(f & kFlagSkip)) {
                        const bool closing = (f & kFlagInfo) != 0;
                        const uint32_t last = (uint32_t)a[3].src;   // closing: source | target << 16
                        // the target, opaque to the optimiser: for the batches that stay in registers it would
                        // otherwise keep every target's addresses in registers of their own across the time loop
                        auto target = [&]() {
                            uint32_t v = last;
                            asm volatile("" : "+v"(v));
                            return v >> 16;
                        };
                        if constexpr (LINW) {
                            // weights as 2^w: a multiply-add per term in place of the add before the exponential;
                            // arcs of weight zero-bar gather the dump slot (zero-bar) and never raise the maximum
                            lse_add4w(m, sum, gv[0], gv[1], gv[2], gv[3], a[0].w, a[1].w, a[2].w, a[3].w);
                            if (closing) {
                                const int lg = (int)((f >> kFlagLgShift) & 7u);
                                if (lg) group_total(m, sum, lg, lane);
                                const uint32_t tgt = target();
                                const T pre = m + (T)flog2(sum) - c;   // sum == 0 -> -inf
                                const T x = pre + (T)ern[vix[tgt]] * (T)kLog2e;
                                xn[tgt] = x;
                                if (keep_pre) bn[tgt] = pre;
                                wmax = tmax(wmax, x);
                                m = (T)kNegBig;
                                sum = 0.0f;
                            }
                            return;
                        }
                        const T x0 = gv[0] + (T)a[0].w, x1 = gv[1] + (T)a[1].w, x2 = gv[2] + (T)a[2].w, x3 = gv[3] + (T)a[3].w;
                        if constexpr (TROP) {
                            // (+) = max: keep the largest term and the state it came from (the first of equal terms)
                            auto take = [&](T x, int s) {
                                if (x > m) { m = x; arg = s; }
                            };
                            take(x0, a[0].src);
                            take(x1, a[1].src);
                            take(x2, a[2].src);
                            take(x3, (int)(last & 0xffffu));
                            if (closing) {
                                const int lg = (int)((f >> kFlagLgShift) & 7u);
                                if (lg) group_best(m, arg, lg, lane);
                                const uint32_t tgt = target();
                                const T x = (m - c) + emitted(ern[vix[tgt]]);
                                xn[tgt] = x;
                                bpn[tgt] = (uint16_t)(arg >> kSrcShift);
                                wmax = tmax(wmax, x);
                                m = kNegInf;
                                arg = 0;
                            }
                        } else {
                            lse_add4(m, sum, x0, x1, x2, x3);
                            if (closing) {   // the rows' sums are complete
                                const int lg = (int)((f >> kFlagLgShift) & 7u);
                                if (lg) group_total(m, sum, lg, lane);   // the row's arcs were spread over 2^lg lanes
                                const uint32_t tgt = target();
                                const T pre = m + (T)flog2(sum) - c;   // sum == 0 -> -inf
                                const T x = pre + (T)ern[vix[tgt]] * (T)kLog2e;
                                xn[tgt] = x;
                                if (keep_pre) bn[tgt] = pre;
                                wmax = tmax(wmax, x);
                                m = (T)kNegBig;
                                sum = 0.0f;
                            }
                        }
                    }
                };
                auto rflag = [&](int q) { return ((q < 4 ? rflag0 : rflag1) >> (8 * (q & 3))) & 0xffu; };
                const uint32_t fw_first = n_iter > 0 ? (uint32_t)__builtin_amdgcn_readlane(fwv0, 0) : 0u;
                auto is_stacked = [&](uint32_t f) { return (f & (kFlagDual | kFlagQuad)) != 0; };
                gather(g[0], res[0], vbase, is_stacked(rflag(0)));
                unrolled([&](auto qc) {
                    constexpr int q = decltype(qc)::value;
                    if (q < n_res) {   // (a small graph fills only the first of them: the padding behind is not walked)
                        if constexpr (q + 1 < NRES)
                            fold(std::bool_constant<(q < kMaxStacked)>{}, rflag(q), res[q], g[q % GB], g[(q + 1) % GB], res[q + 1],
                                 q + 1 < kMaxStacked && is_stacked(rflag(q + 1)), q + 1 < n_res);
                        else
                            fold(std::bool_constant<(q < kMaxStacked)>{}, rflag(q), res[q], g[q % GB], g[(q + 1) % GB], ring[0], false, n_iter > 0);
                    }
                }, std::make_integer_sequence<int, NRES>{});
                uint32_t fw = fw_first;
                prio(std::integral_constant<int, 2>{});
                for (int it = 0; it < n_iter; ++it) {
                    if (it == (n_iter + 1) / 2) prio(std::integral_constant<int, 1>{});
                    // flags of the next iteration (its first byte belongs to the batch after this iteration's last)
                    const int itn = it + 1 < n_iter ? it + 1 : it;
                    const uint32_t fwn =
                        itn < kWave ? __builtin_amdgcn_readlane(fwv0, itn) : __builtin_amdgcn_readlane(fwv1, itn - kWave);
#pragma unroll
                    for (int j = 0; j < kRing; ++j) {
                        load_from(ring[(j + kRing - 1) % kRing], rp);
                        if (j == 0 && it + 1 == n_iter) rp = rp0;   // that was the part's last batch
                        else rp += 2 * kWave;
                        __builtin_amdgcn_sched_barrier(0);
                        fold(std::false_type{}, (fw >> (8 * j)) & 0xffu, ring[j], g[(NRES + j) % GB], g[(NRES + j + 1) % GB], ring[(j + 1) % kRing], false,
                             j + 1 < kRing || it + 1 < n_iter);
                    }
                    fw = fwn;
                }
                put_max(i, wmax);
                lds_barrier();
            };
            if constexpr (XF != 0) {
                for (int i = 1; i < Ts; i += 2) {
                    step(i, std::integral_constant<int, 0>{});
                    if (i + 1 < Ts) step(i + 1, std::integral_constant<int, 1>{});
                }
            } else {
                for (int i = 1; i < Ts; ++i) step(i, (i - 1) & 1);
            }
        }

        // ---- last frame: write it out, close log Z with the end weights
        const int last = (Ts - 1) & 1;
        const T *xl = xb + last * Xs;
        if (io_wave) write_row(frame(Ts - 1), keep_pre ? bh + last * Xs : xl);
        if (TROP) {   // the last vector and its shift, for the kernel that joins the two halves: without its largest entry, or
                      // the other half's entries would be lost in it where this frame's emissions are some large mask
            if (io_wave && Ts >= 2) write_bp(Ts - 1, bpb + last * Xs);
            const T M = get_max(Ts - 1);
            const T c = (M == kNegInf) ? (T)0 : M;
            T *mrow = (T *)R.mid + (size_t)b * R.mid_ld;
            for (int k = tid; k < K; k += NT) mrow[k] = xl[k] - c;
            for (int k = tid; k < nC; k += NT) mrow[P.Kcap + k] = xl[P.Kcap + k] - c;
            if (io_wave && lane == 0) R.mid_off[b] = csum + (double)c;
        } else if (R.logz) {
            T m = (T)kNegBig;
            float s = 0.0f;
            for (int k = tid; k < K; k += NT) lse_add(m, s, xl[k] + (T)R.obound[k0 + k]);
            for (int j = tid; j < sd.n_cdesc; j += NT) {   // clones end with their state's weight
                const CloneDesc cd = cdesc[j];
                for (int i = 0; i < cd.count; ++i) lse_add(m, s, xl[P.Kcap + cd.first + i] + (T)R.obound[k0 + cd.state]);
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) lse_merge(m, s, (T)__shfl_xor(m, o, 64), __shfl_xor(s, o, 64));
            T *rm = red + 2 * NW, *rs = rm + NW;
            if (lane == 0) { rm[wave] = m; rs[wave] = (T)s; }
            __syncthreads();
            if (io_wave && lane == 0) {   // the lane that holds the sum of the offsets
                m = rm[0]; s = (float)rs[0];
                for (int w = 1; w < NW; ++w) lse_merge(m, s, rm[w], (float)rs[w]);
                R.logz[b] = (csum + (double)m + (double)flog2(s)) * kLn2;
            }
        }
    } else if (tid == 0) {
        if (!TROP && R.logz) R.logz[b] = -INFINITY;
    }

    // ---- padded frames
    if (R.fill_pad) {
        if (out_f)
            for (int f = Tn; f < P.N; ++f) {
                float *orow = out_f + (size_t)f * out_ld;
                for (int k = tid; k < K; k += NT) orow[k] = -INFINITY;
            }
        if (off_seq)
            for (int f = Tn + tid; f < P.N; f += NT) off_seq[f] = 0.0;
    }

}

// ---------------------------------------------------------------------------
// The same recursions carried in the probability domain (the matrix products of Eq. 4-5, rescaled at every step;
// the results handed out are those of Eq. 13-14).  For large shared graphs with float vectors.
//
// The vector in LDS holds P[k] = 2^(log2 of the true value - offset), the offset accumulated per sequence, so an
// arc costs one LDS gather and one multiply-add (the plan carries 2^w) and a row one exponential (its emission)
// instead of one exponential per arc.  At every step the vector is rescaled by the power of two that brings the
// previous step's largest entry to [2^bias, 2^(bias + 1)) (exact), and the emissions of a frame enter relative to
// the frame's largest emission over all pdfs (any scale serves).  bias is chosen per graph and direction so that no
// row sum can overflow (from the largest sum of weights of a row).
//
// The plan (fb_pstream.cpp).  Each arc-walking wave has a list of units - two arcs per lane in three registers - most
// of which stay in registers for the whole time loop (the rest cycles through a small ring fed from L2), a bit per
// unit that says whether a slice of rows ends there, and a register per slice that says, per lane, where the
// lane's sum goes and which emission it takes.  The order of the arcs in a lane and of the rows in a slice has been
// chosen on the host so that the 32 lanes of half a wave gather from different banks.
//
// Range guard.  A float holds what lies within 2^-126 of the scale; the log form holds everything.  An entry that is
// not the semiring zero must not come to lie below `dim`, the value under which its product with the graph's smallest
// weight could be flushed to zero.  A lane keeps the smallest entry it has written in a step for a row whose sum is
// above zero (an entry that an emission factor too small for a float has turned into zero included); if that is
// below `dim`, or if the step's largest entry falls too far for the next rescaling to be a float, the workgroup gives
// the sequence up (returns false) and its caller runs it again from the first frame in the log form.  Every sum a
// completed run has formed is therefore exact to rounding.  The give-up travels through the step maximum the waves
// exchange anyway: a lane that sees such a state reports +inf as its maximum.
//
// What leaves the kernel: the vectors as they are kept (RecDir::out_linear, for the gradient kernel) or, in the
// form of the other kernel, normalised rows as logarithms (the wave that closes a row stages its logarithm; the
// data-moving wave copies rows out either way); shifts and log Z as there.
// LDS: xb, the previous / current vector, kXsFixed floats each at addresses 0 and kXbStride; bh 2 x kXsFixed behind
// them (rows on their way out that are not the vector itself: beta before the emission is applied, or either
// direction's rows as logarithms; absent otherwise); red kProbWords floats (3 and 7 scratch of the first frame, 4 the
// largest emission of the first, later of the last frame, 5 that of the second, behind them the slots: the leaky mode's
// sums, at the end the last reduction); er 3 x Es floats, Es = D + 3 rounded up to 4: the emissions as given of the frame in use and of the next two, entry D = -inf (what the dump slot "emits"), in
// the last two places the row's largest emission in log2 units and the largest entry of the vector of its step.
// ---------------------------------------------------------------------------
__device__ unsigned int g_linear_restarts;   // diagnostic: sequences (x directions) given up by linear_run since the library was loaded

typedef uint32_t close_vector_t __attribute__((ext_vector_type(kPMaxClose + 1)));

// LEAKY: the same recursion for the leaky-HMM of the graph (fb_leaky_posteriors), whose transition matrix is
// (I + leak 1 pi^T) T.  The rank-one term stays apart from the sparse one and needs one number of the previous vector:
//   forward   row j gets leak sum_k(x[k]) q[j],  q = T^t pi            (sum weights 1, share of a row q)
//   backward  row i gets leak sum_k(q[k] x[k])                          (sum weights q, share of a row 1)
// so a lane adds up what it writes (times its sum weight), a wave leaves its sum in a slot, and every wave adds the
// slots of the previous step up in the same order when a step starts.  q sits in LDS by target; the entry of the slice
// that closes next is asked for when the one before it has closed.  A clone takes no share of its own (its sign bit
// says so).  A run that leaves the range gives up as below; its caller redoes that sequence with the plain kernel.
// LOG: rows leave as logarithms.  FEW (kPFew, kPFewMost or 0): no wave has more than that many units, so all of them stay in
// registers, nothing is re-read, and the registers that leaves take gathers further ahead.
// States that get nothing from the rest of the graph and so may fall ever further behind it (PStreamDev::apart) are run by the
// data-moving wave, once an entry of the vector has come to lie below the range, a lane a state, in the log form: their entries are what a
// float holds of them, zero below its range.  Such an entry is lost, and so is one of which more than 2^-24 came from lost ones: the rows that leave lack mass that it stands for.
// A lost entry may not matter any more - its share in the sum of any state of the rest, in each frame, and at the end in log Z, below
// 2^-24 - or the run gives up as below.  (Shares of several frames add up: of a posterior at most the number of frames times 2^-24 is missing.)
// TROP: the best path (fb_viterbi).  The vector is scores in log2 units, the largest of the step before taken off at every step, the units
// carry weights in log2 units, a row is the largest of its terms: two additions and one maximum of three a unit.  Which arc
// attains it is not kept: rows leave as they are, and fb_best_trace_kernel finds it anew for the one row a frame that the
// path takes.  A direction goes half way (path_middle); there is no range to leave.
template <bool LEAKY, bool LOG, int FEW, bool TROP = false, bool APART = false>
__device__ __forceinline__ bool linear_run(const RecParams &P, const int b, const int which, double *lds_raw)
{
    constexpr int NW = kNWShared, XF = kXsFixed, R = FEW ? FEW : kPResident;
    constexpr int NT = NW * kWave, NC = NW - 1;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool io_wave = wave == NC;
    const RecDir &R_ = P.dir[which];
    const PStreamDev &S = R_.prob;
    const bool bwd = R_.backward != 0;
    const int K = P.Kcap, nC = S.Ccap;
    const int Tn = min(max(P.lengths[b], 0), P.N);
    const int Ts = !TROP || Tn <= 0 ? Tn : bwd ? Tn - path_middle(Tn) : path_middle(Tn) + 1;   // frames this direction visits
    constexpr float kNone = TROP ? -INFINITY : 0.0f;   // zero-bar
    const int nE = P.D;
    const int nX = K + nC + 1;                   // states, clone slots, dump slot
    // the two buffers of the vector in use lie kXbStride bytes apart, at least a buffer's length: a source or a target is
    // an offset into a buffer, and which buffer is the constant offset of an LDS instruction, 16 bits
    constexpr int Xs = kXbStride / 4;
    static_assert(kXbStride >= XF * 4 && kXbStride < 0x10000, "buffer stride");
    const int Es = prob_row_floats(P.D);
    if (Tn <= 0) return false;                   // (nothing to run: the log form writes the empty results)

    float *xb = (float *)lds_raw;
    // rows on their way out that are not the vector itself: beta before the emissions are applied (backward), and
    // either direction's rows as logarithms when that is the form they leave in; two buffers that follow each other,
    // present only when used
    constexpr bool log_rows = LOG;
    const bool staged = !TROP && (bwd || log_rows);
    const int XL = LEAKY ? (nX + 3) & ~3 : XF;   // floats of a buffer behind the first (leaky: q needs the room)
    float *bh = xb + Xs + XL;
    float *red = staged ? bh + 2 * XL : bh;
    float *slots = red + 8;
    float *qt = red + kProbWords;                // leaky only: q by target
    float *er = LEAKY ? qt + XL : red + kProbWords;
    float *emaxw = red + 4;

    const float *em_seq = P.emis + (size_t)b * P.N * P.D;
    const size_t out_ld = (size_t)(R_.out_ld ? R_.out_ld : K);
    float *out_row0 = R_.out ? (float *)R_.out + (size_t)b * P.N * out_ld : nullptr;
    double *off_seq = R_.off ? R_.off + (size_t)b * P.N : nullptr;
    auto frame = [&](int i) { return bwd ? Tn - 1 - i : i; };
    // the word of step i: the largest entry of its vector, in the last place of the emission row that is in use then (cleared
    // when that row is made ready, read for the last time before the next frame's row is made ready there)
    auto step_word = [&](int i) { return er + (i % 3) * Es + Es - 1; };
    const int kLinBias = S.bias - (LEAKY ? kLeakyBiasDrop : 0);
    const float kLinDimP = S.dim;
    // A step maximum, as its bits: it is never negative, and the bits of such floats have their order.  The run cannot go on
    // from one that is not finite: a lane has given up (+inf).  Below mx_floor the vector fell more than 126 binary orders in
    // one step and its rescaling would not be a float: the data-moving wave then gives up for the step that follows.
    const uint32_t mx_floor = (uint32_t)max(kLinBias - 126 + 127, 1) << 23;
    // The power of two that brings mx (0 or >= mx_floor) to [2^bias, 2^(bias + 1)).  (For 0 a negative number, which leaves
    // every sum of that step, all zero, a zero.)
    const uint32_t sc_top = (uint32_t)(254 + kLinBias) << 23;
    auto rescale = [&](uint32_t mx) { return __uint_as_float(sc_top - (mx & 0x7f800000u)); };

    // ---- duties of the data-moving wave
    // a frame's emissions -> LDS, 16 bytes a lane where the row allows it; the lane's address is formed once and every
    // piece but the last is loaded by all lanes
    auto stage = [&](int f, float *dst) {
        const float *row = em_seq + (size_t)f * P.D;
        typedef const __attribute__((address_space(1))) void gvoid;
        typedef __attribute__((address_space(3))) void lvoid;
        if ((P.D & 3) == 0 && ((uintptr_t)row & 15) == 0) {
            const float *mine = row + 4 * lane;
            int e0 = 0;
            for (; e0 + 4 * kWave <= nE; e0 += 4 * kWave) __builtin_amdgcn_global_load_lds((gvoid *)(mine + e0), (lvoid *)(dst + e0), 16, 0, 0);
            if (e0 + 4 * lane < nE) __builtin_amdgcn_global_load_lds((gvoid *)(mine + e0), (lvoid *)(dst + e0), 16, 0, 0);
        } else {
            const float *mine = row + lane;
            int e0 = 0;
            for (; e0 + kWave <= nE; e0 += kWave) __builtin_amdgcn_global_load_lds((gvoid *)(mine + e0), (lvoid *)(dst + e0), 4, 0, 0);
            if (e0 + lane < nE) __builtin_amdgcn_global_load_lds((gvoid *)(mine + e0), (lvoid *)(dst + e0), 4, 0, 0);
        }
    };
    auto staged_wait = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    // The same for the requests of the step before, where at least `later` memory operations were issued behind them (those
    // of a wave complete in order): the later ones need not have arrived, nor at the step's barrier.  (6000 states, one
    // direction with rows over 540 frames: 2295 us waiting for the stores of the step before as well, 2232 us so.)
    auto staged_before = [&](int later) {
        switch (min(later, 60) >> 2) {
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 1: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); break;
        case 5: asm volatile("s_waitcnt vmcnt(20)" ::: "memory"); break;
        case 6: asm volatile("s_waitcnt vmcnt(24)" ::: "memory"); break;
        case 7: asm volatile("s_waitcnt vmcnt(28)" ::: "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(32)" ::: "memory"); break;
        }
    };
    // pieces of 16 bytes a lane: body(constant n, q) for the n <= 8 pieces from piece q on, until all n_pieces are done
    auto in_groups = [&](int n_pieces, auto body) __attribute__((always_inline)) {
        constexpr int U = 8;
        int q = 0;
        for (; q + U <= n_pieces; q += U) body(std::integral_constant<int, U>{}, q);
        const int rest = n_pieces - q;
        unrolled([&](auto rc) __attribute__((always_inline)) {
            constexpr int n = decltype(rc)::value + 1;
            if (rest == n) body(std::integral_constant<int, n>{}, q);
        }, std::make_integer_sequence<int, U - 1>{});
    };
    // stores and requests a step issues at least: pieces that all lanes have, and a frame's emissions
    const int n_row_stores = out_row0 ? K / (4 * kWave) : 0;
    const bool em_pieces16 = (P.D & 3) == 0 && ((uintptr_t)em_seq & 15) == 0;
    const int n_requests = em_pieces16 ? (P.D + 4 * kWave - 1) / (4 * kWave) : (P.D + kWave - 1) / kWave;
    // The largest emission of a staged frame, in log2 units (0 if there is none above zero-bar).  Over all pdfs, whether a
    // state of the graph is tied to them or not: any scale serves.  16 bytes per lane and read (the arc-walking waves keep
    // the LDS queue full: few, wide reads).  (The factors 2^(emission - largest) are raised where a row closes.  Raised here
    // as well, an exponential per pdf and not per state, a step of 3022 states is 1 % faster with 84 pdfs, but one of 6000
    // states 9 % slower with 3000, and one of 2000 states 7 %: this wave is then what the others wait for.)
    auto last_piece = [&](const float *row, int e0) {
        const int e = e0 + 4 * lane;
        float4 v = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if (e < nE) {
            v = *(const float4 *)(row + e);
            v.y = e + 1 < nE ? v.y : -INFINITY;
            v.z = e + 2 < nE ? v.z : -INFINITY;
            v.w = e + 3 < nE ? v.w : -INFINITY;
        }
        return v;
    };
    auto emax_of = [&](const float *row) {
        float m = -INFINITY;
        const float4 *r4 = (const float4 *)row + lane;
        const int n_full = nE / (4 * kWave);
        in_groups(n_full, [&](auto nc, int q) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            float4 v[n];
#pragma unroll
            for (int u = 0; u < n; ++u) v[u] = r4[(q + u) * kWave];
#pragma unroll
            for (int u = 0; u < n; ++u) m = tmax3(tmax3(m, v[u].x, v[u].y), v[u].z, v[u].w);
        });
        const float4 v = last_piece(row, n_full * 4 * kWave);
        m = tmax3(tmax3(m, v.x, v.y), v.z, v.w);
        m = lane_value(wave_max_last(m), kWave - 1) * (float)kLog2e;
        return m > -INFINITY ? m : 0.0f;
    };
    const CloneDesc *cdesc = S.clones;
    // a finished vector -> global memory, coalesced; a cloned state leaves as the sum of its clones.  Either as it is
    // (RecDir::out_linear: the reader has the offsets and the scale) or as log2 of (entry x 2^-bias) x out_scale, the
    // exponent and the mantissa taken apart first so that neither an entry far below the scale is lost nor the
    // entries near it are rounded at the magnitude of the bias.
    constexpr bool out_lin = !LOG;
    auto log2_of = [&](float v) {
        const float e = (float)(__builtin_amdgcn_frexp_expf(v) - kLinBias);   // (v = 0: -inf comes from the mantissa)
        return e + flog2(__builtin_amdgcn_frexp_mantf(v));
    };
    auto to_log = [&](float v) { return log2_of(v) * R_.out_scale; };
    // (rows that leave as logarithms were staged in that form by the waves that formed them: a plain copy either way)
    auto write_row = [&](int f, const float *srcv) {
        if (!out_row0) return;
        float *orow = out_row0 + (size_t)f * out_ld;
        // (streaming stores: the row is read again much later, by another kernel, and what it would push out of L2 is the arc
        // plan every workgroup re-reads at every step.  Pieces that all lanes have go out without a mask, through a buffer
        // descriptor: an instruction each; with a mask and an address per store this wave took 200 - 280 clocks a piece and
        // was what a step waited for.  The piece's offset is the lane's, not the scalar one: behind a 16-byte store with a scalar
        // offset register the compiler sees no need for a pause before the data registers are written again, and this chip
        // then stored the new value in the first word of a quarter of the lanes.)
        typedef float f4 __attribute__((ext_vector_type(4)));
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
        const f4 *s4 = (const f4 *)srcv + lane;
        const int n_full = K / (4 * kWave);
        auto dst = __builtin_amdgcn_make_buffer_rsrc((void *)orow, 0, K * 4, 0x00027000);
        const int lane16 = lane * 16;
        constexpr int kStreaming = 2;
        in_groups(n_full, [&](auto nc, int q) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            f4 v[n];
#pragma unroll
            for (int u = 0; u < n; ++u) v[u] = s4[(q + u) * kWave];
#pragma unroll
            for (int u = 0; u < n; ++u) asm volatile("" : "+v"(v[u]));   // every read stays in front of the stores
#pragma unroll
            for (int u = 0; u < n; ++u) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v[u]), dst, lane16 + (q + u) * kWave * 16, 0, kStreaming);
        });
        const int at = n_full * 4 * kWave + 4 * lane;   // the last states, fewer than 256
        if (at < K) {
            const f4 v = s4[n_full * kWave];
            // (a padded row may take up to 3 values that lie behind the states)
            if (at + 3 < K || ((out_ld & 3) == 0 && (size_t)(at + 4) <= out_ld)) {
                __builtin_nontemporal_store((f4u)v, (f4u *)(orow + at));
            } else {
                orow[at] = v.x;
                if (at + 1 < K) orow[at + 1] = v.y;
                if (at + 2 < K) orow[at + 2] = v.z;
            }
        }
        for (int j = lane; j < S.n_clones; j += kWave) {   // stores of one wave to one address keep their order
            const CloneDesc cd = cdesc[j];
            if (out_lin) {
                float t = srcv[cd.state];
                for (int i = 0; i < cd.count; ++i) t = TROP ? tmax(t, srcv[K + cd.first + i]) : t + srcv[K + cd.first + i];
                orow[cd.state] = t;
            } else {   // logarithms (scaled by out_scale, which is positive): the (+)-sum of the clones
                float m = srcv[cd.state];
                for (int i = 0; i < cd.count; ++i) m = tmax(m, srcv[K + cd.first + i]);
                float t = 0.0f;
                if (m > -INFINITY) {
                    const float inv = 1.0f / R_.out_scale;
                    t = fexp2((srcv[cd.state] - m) * inv);
                    for (int i = 0; i < cd.count; ++i) t += fexp2((srcv[K + cd.first + i] - m) * inv);
                }
                orow[cd.state] = m > -INFINITY ? m + flog2(t) * R_.out_scale : m;
            }
        }
    };
    // what the readers of a row get beside it: log2 of the true row = log2 of the stored row + cum (in the linear
    // form the stored row still carries the scale 2^bias)
    const double cum_shift = out_lin ? (double)kLinBias : 0.0;

    // ---- first frame of this direction: the start weights and the frame's emissions, relative to their maximum
    if (tid < 3) {
        *step_word(tid) = kNone;
        er[tid * Es + P.D] = -INFINITY;   // what the dump slot "emits" (staging never writes there): its entry stays zero
    }
    if (tid < 8) red[tid] = (tid == 7 || tid == 3) ? -INFINITY : 0.0f;
    if constexpr (LEAKY) {
        for (int k = tid; k < nX; k += NT) qt[k] = R_.rank1[k];
        if (tid < 2) slots[tid * NW + NC] = 0.0f;   // (the data-moving wave writes no rows)
    }
    __syncthreads();
    if (io_wave) {
        stage(frame(0), er);
        if (Ts > 1) stage(frame(1), er + Es);
        staged_wait();
        const float e0 = TROP ? 0.0f : emax_of(er);
        const float e1 = !TROP && Ts > 1 ? emax_of(er + Es) : 0.0f;
        if (lane == 0) { emaxw[0] = e0; emaxw[1] = e1; }
        if (Ts > 1 && lane == 0) er[Es + Es - 2] = e1;
        if (Ts > 2) stage(frame(2), er + 2 * Es);   // lands while step 1 runs
    }
    __syncthreads();
    const float emx0 = emaxw[0];
    if constexpr (!TROP) {
        float ymax = -INFINITY, smax = -INFINITY;
        for (int k = tid; k < K; k += NT) {
            const float s = R_.bound[k];
            ymax = tmax(ymax, s + fmaf(er[P.pdf[k]], (float)kLog2e, -emx0));
            smax = tmax(smax, s);
        }
        ymax = wave_max_last(ymax);
        smax = wave_max_last(smax);
        if (lane == kWave - 1) {
            lds_raise(red + 7, ymax);
            lds_raise(red + 3, smax);
        }
    }
    lds_barrier();
    const float M0 = TROP ? 0.0f : red[7];
    // log2 of the first vector = log2 of its entries + base0 (+ the emission maximum).  The largest entry goes to
    // 2^bias; backward, the row that leaves is the start weights before the frame's emissions, which lie above the
    // vector by what the best state's emission lacks to the frame's largest: the scale is held back as far as that
    // row needs to stay a float (the vector's entries are then smaller, and below the range the run gives up as ever).
    float base0 = M0 > -INFINITY ? M0 - (float)kLinBias : 0.0f;
    if (!TROP && bwd && M0 > -INFINITY) base0 = tmax(base0, red[3] - 126.0f);
    float wmax = kNone, wsum = 0.0f;
    for (int k = tid; k < K; k += NT) {
        const float s = R_.bound[k];
        if constexpr (TROP) {
            // (the backward recursion ends before the emission of its last frame, which may be this one)
            const float x = bwd && Ts == 1 ? s : fmaf(er[P.pdf[k]], (float)kLog2e, s);
            xb[k] = x;
            wmax = tmax(wmax, x);
            continue;
        }
        const float y = s + fmaf(er[P.pdf[k]], (float)kLog2e, -emx0) - base0;
        const float px = fexp2(y);
        xb[k] = px;
        if (log_rows) bh[k] = ((bwd ? s - base0 : y) - (float)kLinBias) * R_.out_scale;
        else if (bwd) bh[k] = fexp2(s - base0);
        const bool dim = y > -INFINITY && px < kLinDimP;
        wmax = dim ? INFINITY : tmax(wmax, px);
        if constexpr (LEAKY) wsum = bwd ? fmaf(fabsf(qt[k]), px, wsum) : wsum + px;
    }
    if constexpr (LEAKY) {
        wsum = wave_sum(wsum);
        if (lane == 0) slots[wave] = wsum;
    }
    for (int k = tid; k < nC; k += NT) {   // clones start empty: the state itself holds the start weight
        xb[K + k] = kNone;
        if (staged) bh[K + k] = log_rows ? -INFINITY : 0.0f;
    }
    if (tid == 0) xb[nX - 1] = xb[Xs + nX - 1] = kNone;   // the dump slot holds zero(-bar) in both buffers, always
    wmax = wave_max_last(wmax);
    if (lane == kWave - 1) lds_raise(step_word(0), wmax);
    lds_barrier();

    // offsets: log2 of the true row of step i = log2 of (the row in LDS x 2^-bias: what is written out) + sum_{j <= i} c_j,
    // with c_0 = base0 + bias (+ the emission maximum of the frame, forward) and c_i = -log2(scale of step i) + the
    // emission maximum of frame(i) (forward) or of frame(i - 1) (backward: the row sum of Eq. 14 is taken before the
    // frame's own emission)
    double csum = 0.0;
    bool ok = true;
    // States that may run apart: they begin in the plan like all others, which costs nothing, and are taken out of it where an entry first comes to lie
    // below the range.  All waves see that at the start of step i, in the word of step i - 1; the vector of step i - 2 and its word
    // are still there, and step i - 1 is done once more, the states apart, from those.  (A run that gives up for another reason gives up again there.)
    // A direction of 64 x 100 frames, us, in the log form from the start where the range is left / apart from the first step on / so: 1500
    // states, 5 k arcs, that stay in range 125 / 197 / 130, that leave it 253 / 208 / 183; 6000 states, 60 k arcs 640 / 340 / 341, over 30 frames
    // 257 / - / 122.
    const bool n_apart = APART && S.apart;   // (an instantiation of its own: the code beside the loop costs others 1 %)
    bool apart_on = false;                  // (uniform over the workgroup)
    auto given_up = [&](const float *word) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(*word)) > 0x7f7fffffu; };
    // whether step i - 1 is to be done once more (i: the step that found the word, or behind the last)
    // (not for step 1: the rows without arcs of the first vector are gone when it is looked at)
    auto to_apart = [&](int i, bool found) { return n_apart && !apart_on && i >= 3 && found; };
    // (data-moving wave)
    int ap_state = -1;
    double ap_value = 0.0;
    float ap_floor = 0.0f, ap_top = 0.0f;   // what the next vector's entries may not lie below; the largest lost entry
    uint64_t ap_lost = 0;                   // the lanes whose entries are lost
    if (io_wave) {
        float c = base0 + (float)kLinBias + (bwd ? 0.0f : emx0);
        csum = TROP ? 0.0 : (double)c;
        if (lane == 0) {
            if (off_seq) off_seq[frame(0)] = csum * (double)R_.out_scale;
            if (R_.cum) R_.cum[(size_t)b * P.N + frame(0)] = (float)(csum - cum_shift);
        }
        // ---- the states that run apart: a lane's state, its sources' lanes and weights, its value (log2, true)
        constexpr double kNoValue = -1.0e36;                // (below kNegBig: zero-bar)
        int ap_pdf = 0;
        int32_t ap_src[kApartArcs], ap_tgt[kApartTargets];
        float ap_w[kApartArcs];
        // from the vector x of a step on, whose shift is csum
        auto apart_begin = [&](const float *x) {
            const int32_t *ap = S.apart + lane;
            ap_state = ap[0];
#pragma unroll
            for (int t = 0; t < kApartArcs; ++t) {
                ap_src[t] = ap[(1 + t) * kWave];
                ap_w[t] = __int_as_float(ap[(1 + kApartArcs + t) * kWave]);
            }
#pragma unroll
            for (int t = 0; t < kApartTargets; ++t) ap_tgt[t] = ap[(1 + 2 * kApartArcs + t) * kWave];
            ap_pdf = P.pdf[max(ap_state, 0)];
            const float v = x[max(ap_state, 0)];
            ap_value = ap_state >= 0 && v > 0.0f ? csum + (double)log2_of(v) : kNoValue;
        };
        // the entries that arcs of theirs enter, in x, against what may have been lost on the way there
        auto apart_check = [&](const float *x, float *word) {
            float low = INFINITY;
#pragma unroll
            for (int t = 0; t < kApartTargets; ++t)
                if (ap_tgt[t] >= 0) low = tmin(low, x[ap_tgt[t]]);
            if (__any(low < ap_floor) && lane == kWave - 1) lds_raise(word, INFINITY);
        };
        auto apart_step = [&](int i, const float *row, float *word, float minus_log2_scale) {
            const int nxt = i & 1;
            if (ap_floor > 0.0f) apart_check(xb + (nxt ^ 1) * Xs, word);
            // (for vector i: its sums take the lost entries of vector i - 1, times the step's scale)
            ap_floor = !ap_lost ? 0.0f : fexp2(tmin(tmax(-minus_log2_scale + S.apart_gain + 24.0f + flog2(tmax(kLinDimP, ap_top)), -126.0f), 127.0f));
            double v[kApartArcs], top = kNoValue;
#pragma unroll
            for (int t = 0; t < kApartArcs; ++t) {
                v[t] = __shfl(ap_value, max(ap_src[t], 0), kWave) + (double)ap_w[t];
                v[t] = ap_src[t] >= 0 ? v[t] : kNoValue;
                top = fmax(top, v[t]);
            }
            float sum = 0.0f;
#pragma unroll
            for (int t = 0; t < kApartArcs; ++t) sum += fexp2((float)(v[t] - top));
            const double all = top + (double)flog2(sum), now = all + (double)row[ap_pdf] * kLog2e;
            bool lost = false;
#pragma unroll
            for (int t = 0; t < kApartArcs; ++t) lost = lost || (ap_src[t] >= 0 && ((ap_lost >> (ap_src[t] & 63)) & 1u) && !(v[t] < all - 24.0));
            const bool live = ap_state >= 0 && !(now < (double)kNegBig);   // (a NaN is)
            ap_value = live ? now : kNoValue;
            const double at = ap_value - csum, e = __builtin_rint(at + (double)kLinBias);
            const float x = live ? ldexpf(fexp2((float)(at + (double)kLinBias - e)), (int)fmin(fmax(e, -1000.0), 1000.0)) : 0.0f;
            if (ap_state >= 0) {
                xb[nxt * Xs + ap_state] = x;
                if (staged) bh[nxt * XL + ap_state] = live ? (float)at * R_.out_scale : -INFINITY;
            }
            lost = live && (lost || x < kLinDimP);
            ap_lost = __ballot(lost);
            ap_top = lane_value(wave_max_last(lost ? x : 0.0f), kWave - 1);
            const float most = wave_max_last(x);
            // (a lost entry of a state that is alive in the first frames only: what it enters is not looked at)
            const bool odd = S.apart_lasting < kWave && (ap_lost >> S.apart_lasting) != 0;
            if (lane == kWave - 1) lds_raise(word, odd ? INFINITY : most);
        };
        float e_prev = emx0, e_cur = Ts > 1 ? emaxw[1] : 0.0f;   // the largest emission of frame i - 1 and of frame i
        float *row_a = er, *row_b = er + Es, *row_c = er + 2 * Es;   // rows of frame i - 1 (from step i on: i + 2), i, i + 1
        double csum_before = 0.0;   // the shift of the step before
        // back to the start of step i - 1 from that of step i, the emissions of frame i + 2 asked for and row i - 1 stored or not
        auto back = [&](int i) {
            staged_wait();          // (a row that is stored again comes behind the one under way)
            stage(frame(i - 1), row_a);
            csum = csum_before;
            e_cur = e_prev;
            apart_begin(xb + (i & 1) * Xs);
            __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0), as the compiler knows: the loop's waits count its own loads only
            lds_barrier();          // every wave has read the word
            if (lane == 0) row_a[Es - 1] = kNone;
            lds_barrier();
            float *const t = row_c;
            row_c = row_b;
            row_b = row_a;
            row_a = t;
            apart_on = true;
        };
        int found_at = Ts;          // the step that found a word that ends the run
        for (int i = 1; i < Ts; ++i) {
            const int cur = (i - 1) & 1;
            const float mxv = row_a[Es - 1];
            const bool more = i + 2 < Ts;
            // (the word of step i - 1 lies behind what is staged)
            if (more) stage(frame(i + 2), row_a);   // buffer of frame i-1: no longer read
            write_row(frame(i - 1), staged ? bh + cur * XL : xb + cur * Xs);
            const uint32_t mx = (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(mxv));
            if (!TROP && mx > 0x7f7fffffu) {
                if constexpr (APART) found_at = i;
                ok = false;
                break;
            }
            const float nls = TROP ? (mxv > -INFINITY ? mxv : 0.0f) : mx > 0u ? (float)((int)(mx >> 23) - 127 - kLinBias) : 0.0f;   // minus log2 of the step's scale
            c = TROP ? nls : nls + (bwd ? e_prev : e_cur);
            if constexpr (APART) csum_before = csum;
            csum += (double)c;
            if (lane == 0) {
                if (off_seq) off_seq[frame(i)] = csum * (double)R_.out_scale;
                if (R_.cum) R_.cum[(size_t)b * P.N + frame(i)] = (float)(csum - cum_shift);
            }
            if (!TROP && mx > 0u && mx < mx_floor && lane == kWave - 1) lds_raise(row_b + Es - 1, INFINITY);
            e_prev = e_cur;
            if (i + 1 < Ts) {
                staged_before(n_row_stores + (more ? n_requests : 0));   // frame i+1, requested a whole step ago, is in LDS
                if constexpr (!TROP) e_cur = emax_of(row_c);
                if (lane < 2) row_c[Es - 2 + lane] = lane ? kNone : e_cur;   // and the word of step i + 1 starts empty
            }
            if (LEAKY && lane == 0) slots[(i & 1) * NW + NC] = 0.0f;
            float *const t = row_a;
            row_a = row_b;
            row_b = row_c;
            row_c = t;
            lds_barrier();   // (the row's stores and the emissions asked for go on)
        }
        // The same loop with the states apart.  (A loop of its own: the registers they keep cost steps without them 8 to 13 % on small plans; and both
        // as calls of one closure the compiler no longer split the loop by what does not change in it, up to 8 % on plans of up to 16 units.)
        if constexpr (APART) {
            if (to_apart(found_at, !ok || given_up(row_a + Es - 1))) {
                back(found_at);
                ok = true;
                for (int i = found_at - 1; i < Ts; ++i) {
                    const int cur = (i - 1) & 1;
                    const float mxv = row_a[Es - 1];
                    const bool more = i + 2 < Ts;
                    if (more) stage(frame(i + 2), row_a);
                    write_row(frame(i - 1), staged ? bh + cur * XL : xb + cur * Xs);
                    const uint32_t mx = (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(mxv));
                    if (mx > 0x7f7fffffu) { ok = false; break; }
                    const float nls = mx > 0u ? (float)((int)(mx >> 23) - 127 - kLinBias) : 0.0f;
                    csum += (double)(nls + e_cur);   // (forward plans only)
                    if (lane == 0) {
                        if (off_seq) off_seq[frame(i)] = csum * (double)R_.out_scale;
                        if (R_.cum) R_.cum[(size_t)b * P.N + frame(i)] = (float)(csum - cum_shift);
                    }
                    apart_step(i, row_b, row_b + Es - 1, nls);
                    if (mx > 0u && mx < mx_floor && lane == kWave - 1) lds_raise(row_b + Es - 1, INFINITY);
                    e_prev = e_cur;
                    if (i + 1 < Ts) {
                        staged_before(n_row_stores + (more ? n_requests : 0));
                        e_cur = emax_of(row_c);
                        if (lane < 2) row_c[Es - 2 + lane] = lane ? 0.0f : e_cur;
                    }
                    float *const t = row_a;
                    row_a = row_b;
                    row_b = row_c;
                    row_c = t;
                    lds_barrier();
                }
            }
        }
        if (lane == 0) emaxw[0] = e_prev;   // that of the last frame, for log Z
        if (apart_on && ok && ap_floor > 0.0f) apart_check(xb + ((Ts - 1) & 1) * Xs, step_word(Ts - 1));
    } else {
        const PWaveDesc wd = S.waves[wave];
        const int n_units_w = __builtin_amdgcn_readfirstlane(wd.n_units);
        auto uniform64 = [](uint64_t v) {
            return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
                   ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32);
        };
        const uint64_t mask0_w = uniform64(wd.close_mask[0]), mask1_w = uniform64(wd.close_mask[1]), lgs_w = uniform64(wd.lgs);
        // (s1: the second source apart from the first, where registers allow it: an address then needs no instruction)
        constexpr bool kApart = FEW == kPFew;
        struct Unit { uint32_t s, s1; float w0, w1; };
        // Unit u of the wave: three words per lane, read through a buffer descriptor, whose scalar offset is the unit's: a
        // request takes no vector instruction (an address formed from a scalar base and a large constant takes four).
        constexpr int kUnitBytes = 3 * kWave * 4;
        auto units_of = [&](const uint32_t *of) __attribute__((always_inline)) {
            return __builtin_amdgcn_make_buffer_rsrc((void *)(of + (size_t)uniform64((uint64_t)wd.unit_base) * (3 * kWave)), 0,
                                                     max(n_units_w, FEW ? FEW : kPPatterned) * kUnitBytes, 0x00027000);
        };
        auto units = units_of(S.units);
        const int lane12 = lane * 12;
        auto load_unit = [&](Unit &dst, int u) __attribute__((always_inline)) {
            typedef uint32_t u3 __attribute__((ext_vector_type(3)));
            const u3 v = __builtin_amdgcn_raw_buffer_load_b96(units, lane12, u * kUnitBytes, 0);
            dst.s = kApart ? v.x & 0xffffu : v.x;
            dst.s1 = kApart ? v.x >> 16 : 0u;
            dst.w0 = __uint_as_float(v.y);
            dst.w1 = __uint_as_float(v.z);
        };
        // The wave's units in walking order (see kPPatterned): which positions stay in registers, which are re-read.
        // Re-read ("streamed") unit m of a step sits in ring[m % kPRing] and is asked for kPRing - 1 streamed units ahead
        // of its use; the first kPRing - 1 of a step when the step before ends.  Every place that asks does so whatever
        // the wave's unit count (for a unit that is not there, the last one again): the number of loads on their way
        // at any point of the code is then a constant, which is what the waits on them are counted by.
        constexpr int NP = FEW ? FEW : kPPatterned, H = kPHead, NG = NP - R;   // patterned positions, head, re-read ones among them
        static_assert(NP <= 64 && NP % 4 == 0 && (FEW || NG >= kPRing - 1), "close bits of the patterned part in one 64-bit word; blocks of 4");
        constexpr int kQuarter = (NP / 4 + 3) / 4 * 4;   // a priority level for every quarter, in whole blocks
        // the position of the wave's last re-read unit: what a request for a unit behind it asks for again (a wave
        // without any asks for a unit behind its own: never folded, and the plan has room behind every wave)
        int last_spos = p_streamed_pos(0);
        unrolled([&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value;
            if constexpr (!FEW && p_streamed(u)) last_spos = u < n_units_w ? u : last_spos;
        }, std::make_integer_sequence<int, NP>{});
        if (n_units_w > NP) last_spos = n_units_w - 1;
        Unit res[R];   // (units behind the wave's last one are zero words or another wave's: never folded)
        // The lane's close words, picked by the number of the close (uniform).  One vector of nine: picking from a vector of
        // eight is compiled into a chain of seven selects, from a longer one into one indexed register move.
        close_vector_t cwv;
        auto load_plan = [&](const uint32_t *close_words) __attribute__((always_inline)) {
            unrolled([&](auto qc) __attribute__((always_inline)) {
                constexpr int q = decltype(qc)::value, pos = FEW ? q : p_resident_pos(q);
                load_unit(res[q], pos);
            }, std::make_integer_sequence<int, R>{});
#pragma unroll
            for (int c = 0; c < kPMaxClose; ++c) cwv[c] = close_words[((size_t)wd.cw_base + c) * kWave + lane];
            cwv[kPMaxClose] = cwv[0];   // (what is asked for when the last slice has closed)
            // (everything asked for so far has arrived: the waits inside the loop then count the loop's own loads only)
            __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
        };
        load_plan(S.close_words);
        // The steps' code begins so many words behind a line of the 32 bytes that instructions are fetched by, whatever comes before it:
        // where steps are mostly short blocks and jumps, the place alone makes up to a tenth.  At zero to seven words, us a call:
        // LF-MMI of 1163 states, 17 k arcs, 2777 labels, 31 sequences  1065 1062 1059 1080 1084 1152 1063 1047 (1155 where it happened to fall),
        // sums of 1444 states, 20 k arcs, 61 sequences                  878  876  876  879  880  904  908  950,
        // sums of 4830 states, 27 k arcs, 23 sequences, states apart    372  382  364  365  362  363  363  370,
        // LF-MMI of 6000 states, 60 k arcs, 128 sequences              2116 2111 2145 2129 2116 2128 2116 2125.
        constexpr int kWords = FEW && !APART && !TROP ? 2 : 4;
        asm volatile(".p2align 5\n\t.rept %0\n\ts_nop 0\n\t.endr" : : "n"(kWords));
        Unit ring[kPRing];
        // streamed unit m -> its ring place (in the patterned part streamed unit m is position H + 3 m + 2; behind it, unit
        // NP + t is streamed unit NG + t)
        // (a position inside the patterned part is asked for as it is, whatever the wave's unit count: the plan has
        // room for kPPatterned units behind every wave's first; positions behind it are held to the wave's last unit)
        auto request_at = [&](Unit &dst, int u) __attribute__((always_inline)) {
            load_unit(dst, u);
            __builtin_amdgcn_sched_barrier(0);   // keep the issue order: waits count loads in order
        };
        auto request = [&](Unit &dst, int pos) __attribute__((always_inline)) { request_at(dst, min(pos, last_spos)); };
        unrolled([&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value, first = p_streamed_pos(m);
            request_at(ring[m], first);
        }, std::make_integer_sequence<int, FEW ? 0 : kPRing - 1>{});

        // Scalar instructions and branches are what a step is short of: a SIMD issues one in about 5.5 clocks whatever the
        // number of its waves (a plain vector instruction in 2.4), and a step of 3022 states, 51 k arcs took 2900 of them
        // over its 16 waves beside 3200 vector instructions, in 5100 clocks.  Hence: what a step needs of the rotating rows is
        // one running address, and scales and the range guard are vector arithmetic.  (Asked once for every four units whether
        // a slice ends among them, a step takes 700 scalar instructions fewer, but 800 moves more where the two paths meet.)
        uint32_t m_lo = (uint32_t)mask0_w, m_hi = (uint32_t)(mask0_w >> 32), m1_lo = (uint32_t)mask1_w, m1_hi = (uint32_t)(mask1_w >> 32);
        uint32_t lg_lo = (uint32_t)lgs_w;
        int n_units = n_units_w, n_wide = 0;   // slices whose rows take several lanes: the plan has them in front
#pragma unroll
        for (int c = 0; c < kPMaxClose; ++c) n_wide = ((lg_lo >> (3 * c)) & 7u) ? c + 1 : n_wide;
        typedef __attribute__((address_space(3))) float lds_f;
        typedef const __attribute__((address_space(3))) float lds_cf;
        const uint32_t row_bytes = (uint32_t)Es * 4u, row_first = (uint32_t)(uintptr_t)(lds_cf *)er, row_end = row_first + 3u * row_bytes;
        uint32_t row_cur = row_first;   // the emission row of the frame in hand
        uint32_t to_word = row_bytes - 8u;   // of a row: its largest emission, then the word of the step's maximum
        asm volatile("" : "+v"(to_word));   // (a vector register: what is added to it is then no scalar addition)

        // Two steps, one after the other, are two copies of the code: which buffer holds the previous step's vector is then
        // known, and its address is the constant offset of an LDS instruction.  (With the address OR-ed into a source by the
        // instruction that takes the source out of its word, that instruction is one of sub-words, which issue at little
        // more than half the rate.)
        auto step = [&](int i, auto parity) __attribute__((always_inline)) -> bool {
            constexpr int cur = decltype(parity)::value, nxt = cur ^ 1;   // (i - 1) & 1: the buffer of the previous step's vector
            float *xn = xb + nxt * Xs;
            float *bn = bh + nxt * XL;
            // (the workgroup's LDS starts at address 0)
            const uint32_t bn_at = (uint32_t)((Xs + XL) * 4) + (uint32_t)nxt * (uint32_t)(XL * 4);
            // the wave's constants, opaque at every step: what is derived from them is computed where it is used (a
            // scalar instruction or two) instead of being kept in scalar registers that do not exist
            asm volatile("" : "+s"(m_lo), "+s"(m_hi), "+s"(m1_lo), "+s"(m1_hi), "+s"(lg_lo), "+s"(n_units), "+s"(last_spos));
            const float mxv = *(lds_cf *)(uintptr_t)(row_cur + to_word + 4u);
            row_cur += row_bytes;
            row_cur = row_cur == row_end ? row_first : row_cur;
            const uint32_t ern = row_cur;   // the frame's emissions
            const float emx = *(lds_cf *)(uintptr_t)(ern + to_word);
            // the close word in use, and the emission of its rows: asked for when the slice before has closed
            uint32_t cw = cwv[0];
            float pe = *(lds_cf *)(uintptr_t)(ern + (cw >> 16));
            float sc = 1.0f;
            wmax = kNone;
            const bool no_em = TROP && bwd && i == Ts - 1;   // (see the first frame)
            // the smallest entry this lane has written for a row whose sum is above zero, as its bit pattern (which keeps
            // the order of floats that are not negative)
            uint32_t wlow = 0x7f800000u;
            float acc = kNone;
            // leaky: the previous vector's sum (every wave adds the slots in the same order) and the next close's q
            float leaked = 0.0f, q_next = 0.0f, slot = 0.0f;
            if constexpr (LEAKY) {
                slot = slots[cur * NW + (lane & (NW - 1))];
                wsum = 0.0f;
                q_next = *(const float *)((const char *)qt + (cw & 0xffffu));
            }
            int nclose = 0;   // slices closed so far in this step (uniform)
            if (i == cur + 1)   // rows without arcs: zero from the second frame on, in both buffers
                for (int z = tid; z < S.n_zero; z += NC * kWave) {
                    const int k = S.zero_rows[z];
                    xn[k] = kNone;
                    if (staged) bn[k] = log_rows ? -INFINITY : 0.0f;
                }
            // the two values a unit gathers; sources are byte offsets.  (In assembly so that the addresses are formed at every
            // step: left to itself the compiler keeps every resident unit's two in registers of their own.)
            uint32_t low_half = 0xffffu;
            asm volatile("" : "+s"(low_half));
            auto gather = [&](float2 &g, const Unit &un) __attribute__((always_inline)) {
                typedef const __attribute__((address_space(3))) float lds_ct;
                uint32_t lo = un.s, hi = un.s1;
                if constexpr (!kApart)
                    asm volatile("v_and_b32 %0, %3, %2\n\tv_lshrrev_b32 %1, 16, %2" : "=&v"(lo), "=v"(hi) : "v"(un.s), "s"(low_half));
                g.x = *(lds_ct *)(uintptr_t)(lo + (uint32_t)(cur * kXbStride));
                g.y = *(lds_ct *)(uintptr_t)(hi + (uint32_t)(cur * kXbStride));
            };
            // a slice ends: the lanes of a row are added up, the row is rescaled, takes its emission, is stored
            auto close_slice = [&]() __attribute__((always_inline)) {
                const uint32_t tgt = cw & 0xffffu;
                float share = 1.0f;   // (leaky: a row spread over several lanes, all of which hold it, counts once)
                if (__builtin_expect(nclose < n_wide, 0)) {
                    const int lg = (int)((lg_lo >> (3 * nclose)) & 7u);
                    if constexpr (LEAKY) share = __uint_as_float((uint32_t)(127 - lg) << 23);
                    for (int sft = 0; sft < lg; ++sft) {   // the lanes of a row are neighbours: a butterfly over 2^lg lanes (few rows are that long)
                        const float other = __uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ (1 << sft)) << 2, (int)__float_as_uint(acc)));
                        acc = TROP ? tmax(acc, other) : acc + other;
                    }
                }
                cw = cwv[++nclose];
                const float q = q_next;
                if constexpr (LEAKY) {
                    acc = bwd ? acc + ((int)__float_as_uint(q) >= 0 ? leaked : 0.0f) : fmaf(leaked, tmax(q, 0.0f), acc);
                    q_next = *(const float *)((const char *)qt + (cw & 0xffffu));
                }
                if constexpr (TROP) {
                    const float xb_ = acc - sc;   // (sc: what is taken off, here)
                    const float x = no_em ? xb_ : fmaf(pe, (float)kLog2e, xb_);
                    pe = *(lds_cf *)(uintptr_t)(ern + (cw >> 16));
                    *(lds_f *)(uintptr_t)(tgt + (uint32_t)(nxt * kXbStride)) = x;
                    wmax = tmax(wmax, x);
                    acc = kNone;
                    return;
                }
                const float pb = acc * sc;
                const float px = pb * fexp2(fmaf(pe, (float)kLog2e, -emx));
                pe = *(lds_cf *)(uintptr_t)(ern + (cw >> 16));
                if constexpr (LEAKY) wsum = fmaf(bwd ? fabsf(q) * share : share, px, wsum);
                *(lds_f *)(uintptr_t)(tgt + (uint32_t)(nxt * kXbStride)) = px;
                if (staged) {   // (uniform) what leaves the kernel for this row
                    const float o = bwd ? pb : px;
                    *(lds_f *)(uintptr_t)(tgt + bn_at) = log_rows ? to_log(o) : o;
                }
                wmax = tmax(wmax, px);
                wlow = min(wlow, __float_as_uint(pb > 0.0f ? px : INFINITY));
                acc = 0.0f;
            };
            // position u of the patterned part: which registers hold it
            auto unit_at = [&](auto uc) __attribute__((always_inline)) -> Unit {
                constexpr int u = decltype(uc)::value;
                if constexpr (FEW) return res[u];
                else {
                    constexpr int before = p_streamed_before(u);
                    if constexpr (p_streamed(u)) return ring[before % kPRing];
                    else return res[u - before];
                }
            };
            // gathered values of the unit being folded and of the next GD: under load a gather takes a few hundred cycles
            constexpr int GD = FEW ? 7 : 3, NGB = GD + 1;
            static_assert(FEW || (kPRing % NGB == 0 && NG % kPRing == 0 && GD <= H && GD <= kPRing - 1), "buffer names repeat with the ring; the first gathers are of resident units");
            float2 G[NGB];
            unrolled([&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;
                gather(G[u], unit_at(std::integral_constant<int, u>{}));
            }, std::make_integer_sequence<int, GD>{});
            const uint32_t mx = __float_as_uint(mxv);
            if (!TROP && __builtin_expect((uint32_t)__builtin_amdgcn_readfirstlane((int)mx) > 0x7f7fffffu, 0)) return false;   // (the same word in every wave: all of them leave here)
            sc = TROP ? (mxv > -INFINITY ? mxv : 0.0f) : rescale(mx);
            if constexpr (LEAKY) leaked = P.leak * lane_value(row_sum_last(slot), 15);
            // Waves of equal priority are served oldest first, so with one fixed priority the younger waves of a SIMD
            // would do most of their step alone after the older ones have finished theirs.  A wave's priority therefore
            // falls as its step advances, a level for every quarter: whoever has more left goes first.
            __builtin_amdgcn_s_setprio(3);
            // (the units are in order, so nothing follows a unit that is not there; looked at every fourth position)
            auto block = [&](auto self, auto kc) __attribute__((always_inline)) -> void {
                constexpr int u0 = decltype(kc)::value * 4;
                if constexpr (u0 < NP) {
                    if (n_units > u0) {
                        if constexpr (u0 % kQuarter == 0 && u0 > 0) __builtin_amdgcn_s_setprio(3 - u0 / kQuarter);
                        unrolled([&](auto jc) __attribute__((always_inline)) {
                            constexpr int u = u0 + decltype(jc)::value;
                            // a streamed unit: the place of the one before it in the ring is free, the unit kPRing - 1 further on goes there
                            if constexpr (!FEW && p_streamed(u)) {
                                constexpr int m = p_streamed_before(u), ahead = p_streamed_pos(m + kPRing - 1);
                                if constexpr (ahead < NP) request_at(ring[(m + kPRing - 1) % kPRing], ahead);
                                else request(ring[(m + kPRing - 1) % kPRing], ahead);
                            }
                            // (gathered whether the wave has that unit or not - its registers hold valid sources either way -
                            // so that the number of gathers on their way is a constant too)
                            if constexpr (u + GD < NP) gather(G[(u + GD) % NGB], unit_at(std::integral_constant<int, u + GD>{}));
                            else if constexpr (!FEW) gather(G[(u + GD) % NGB], ring[(NG + (u + GD - NP)) % kPRing]);   // the first units behind the patterned part
                            const Unit me = unit_at(std::integral_constant<int, u>{});
                            // (both values of the unit are taken at one point: one wait for the pair instead of one each)
                            asm volatile("" : "+v"(G[u % NGB].x), "+v"(G[u % NGB].y));
                            if constexpr (TROP) {
                                acc = tmax3(acc, G[u % NGB].x + me.w0, G[u % NGB].y + me.w1);
                            } else {
                                acc = fmaf(G[u % NGB].x, me.w0, acc);
                                acc = fmaf(G[u % NGB].y, me.w1, acc);
                            }
                            if constexpr (!FEW || (u & 1)) {   // (slices of pairs of units: PStreamHost::paired)
                                if (__builtin_expect(((u < 32 ? m_lo : m_hi) >> (u & 31)) & 1u, 0)) close_slice();
                            }
                        }, std::make_integer_sequence<int, 4>{});
                        self(self, std::integral_constant<int, decltype(kc)::value + 1>{});
                    }
                }
            };
            block(block, std::integral_constant<int, 0>{});
            // behind the patterned part: streamed units; unit NP + t is streamed unit NG + t; kPRing positions to a round,
            // so that the names of the ring places and of the gather buffers repeat
            static_assert(FEW || NP % NGB == 0, "rounds");
            if constexpr (!FEW) {
                for (int t0 = 0; NP + t0 < n_units; t0 += kPRing) {
    #pragma unroll
                    for (int tt = 0; tt < kPRing; ++tt) {   // (a plain loop: closures inside a loop that stays a loop are not taken apart by the compiler)
                        const int t = t0 + tt;
                        if (NP + t < n_units) {
                            const int mr = NG + tt;   // (t0 is a multiple of kPRing: only tt names the buffers)
                            request(ring[(mr + kPRing - 1) % kPRing], NP + t + kPRing - 1);
                            gather(G[(NP + tt + GD) % NGB], ring[(mr + GD) % kPRing]);
                            asm volatile("" : "+v"(G[(NP + tt) % NGB].x), "+v"(G[(NP + tt) % NGB].y));
                            if (TROP) {
                                acc = tmax3(acc, G[(NP + tt) % NGB].x + ring[mr % kPRing].w0, G[(NP + tt) % NGB].y + ring[mr % kPRing].w1);
                            } else {
                                acc = fmaf(G[(NP + tt) % NGB].x, ring[mr % kPRing].w0, acc);
                                acc = fmaf(G[(NP + tt) % NGB].y, ring[mr % kPRing].w1, acc);
                            }
                            const int at = NP + t;
                            const uint32_t word = at < 32 ? m_lo : at < 64 ? m_hi : at < 96 ? m1_lo : m1_hi;
                            if (__builtin_expect((word >> (at & 31)) & 1u, 0)) close_slice();
                        }
                    }
                }
            }
            // the first streamed units of the next step (every place of the ring is free now)
            unrolled([&](auto mc) __attribute__((always_inline)) {
                constexpr int m = decltype(mc)::value, first = p_streamed_pos(m);
                request_at(ring[m], first);
            }, std::make_integer_sequence<int, FEW ? 0 : kPRing - 1>{});
            // an entry below the range: the run gives up (see above)
            wmax = wave_max_last(!TROP && wlow < __float_as_uint(kLinDimP) ? INFINITY : wmax);
            lds_raise_last(ern + to_word + 4u, wmax);
            if constexpr (LEAKY) {
                wsum = wave_sum_last(wsum);
                if (lane == kWave - 1) slots[nxt * NW + wave] = wsum;
            }
            lds_barrier();
            return true;
        };
        if constexpr (!APART) {
            for (int i = 1; ok && i < Ts; ++i) {
                ok = step(i, std::integral_constant<int, 0>{});
                if (ok && ++i < Ts) ok = step(i, std::integral_constant<int, 1>{});
            }
        } else {
            for (int i = 1;;) {
                while (i < Ts) {
                    if (i & 1) {   // (or the second step of two is the one done once more)
                        ok = step(i, std::integral_constant<int, 0>{});
                        if (!ok || ++i >= Ts) break;
                    }
                    ok = step(i, std::integral_constant<int, 1>{});
                    if (!ok) break;
                    ++i;
                }
                if (!to_apart(i, !ok || given_up(step_word(Ts - 1)))) break;
                --i;
                units = units_of(S.apart_units);
                lds_barrier();
                load_plan(S.apart_close);
                unrolled([&](auto mc) __attribute__((always_inline)) {
                    constexpr int m = decltype(mc)::value, first = p_streamed_pos(m);
                    request_at(ring[m], first);
                }, std::make_integer_sequence<int, FEW ? 0 : kPRing - 1>{});
                row_cur = row_first + (uint32_t)((i - 1) % 3) * row_bytes;
                lds_barrier();
                ok = true;
                apart_on = true;
            }
        }
    }
    if constexpr (TROP) {
        // ---- the last vector, a cloned state's value the largest of its clones', for the kernel that joins the two halves: without its
        // largest entry, or the other half's entries would be lost in it where this frame's emissions are some large mask
        const float mxl = *step_word(Ts - 1), cl = mxl > -INFINITY ? mxl : 0.0f;
        float *xl = xb + ((Ts - 1) & 1) * Xs;
        for (int j = tid; j < S.n_clones; j += NT) {
            const CloneDesc cd = cdesc[j];
            float v = xl[cd.state];
            for (int i = 0; i < cd.count; ++i) v = tmax(v, xl[K + cd.first + i]);
            xl[cd.state] = v;
        }
        __syncthreads();
        float *mrow = (float *)R_.mid + (size_t)b * R_.mid_ld;
        for (int k = tid; k < K; k += NT) mrow[k] = xl[k] - cl;
        if (io_wave && lane == 0) R_.mid_off[b] = csum + (double)cl;
        return true;
    }
    if (apart_on && ok) lds_barrier();   // (the last vector has been looked at)
    // a state below the range in the last step: give up as well (every wave reads the same word)
    if (ok && !(*step_word(Tn - 1) < INFINITY)) ok = false;   // (the last vector is not rescaled: only a lane's give-up counts)
    __builtin_amdgcn_s_setprio(3);
    auto give_up = [&]() {
        // every wave has left the time loop at the same step; nothing of this run may still be on its way to LDS or
        // to the output rows when the log form starts over
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();
        if (!LEAKY && tid == 0) atomicAdd(&g_linear_restarts, 1u);
    };
    if (!ok) {
        give_up();
        return false;
    }

    // ---- last frame: write it out, close log Z with the end weights
    const int last = (Tn - 1) & 1;
    const float *xl = xb + last * Xs;
    if (io_wave) write_row(frame(Tn - 1), staged ? bh + last * XL : xl);
    if (R_.logz) {
        // (the last vector has not been rescaled: its entries x 2^-bias need not be floats)
        float m = kNegBig, s = 0.0f;
        for (int k = tid; k < K; k += NT) lse_add(m, s, log2_of(xl[k]) + R_.obound[k]);
        for (int j = tid; j < S.n_clones; j += NT) {   // clones end with their state's weight
            const CloneDesc cd = cdesc[j];
            for (int i = 0; i < cd.count; ++i) lse_add(m, s, log2_of(xl[K + cd.first + i]) + R_.obound[cd.state]);
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) lse_merge(m, s, __shfl_xor(m, o, 64), __shfl_xor(s, o, 64));
        float *rm = slots, *rs = rm + NW;
        const float em_last = emaxw[0];
        if (lane == 0) { rm[wave] = m; rs[wave] = s; }
        __syncthreads();
        if (io_wave && lane == 0) {   // the lane that holds the sum of the offsets
            m = rm[0]; s = rs[0];
            for (int w = 1; w < NW; ++w) lse_merge(m, s, rm[w], rs[w]);
            // backward: the vector of the last step still lacks the scale of its frame's emissions
            R_.logz[b] = (csum + (bwd ? (double)em_last : 0.0) + (double)m + (double)flog2(s)) * kLn2;
        }
        if (apart_on) {   // (64 states at most, each no more than the largest)
            if (io_wave && ap_lost) {
                const double share = (ap_lost >> lane) & 1u ? ap_value + (double)R_.obound[ap_state] : -1.0e36;
                const double most = wave_max(share) + 6.0, all = lane_value(csum + (double)m + (double)flog2(s), 0);
                if (lane == 0 && !(most < all - 24.0)) red[6] = 1.0f;
            }
            __syncthreads();
            if (red[6] != 0.0f) {
                give_up();
                return false;
            }
        }
    }
    // ---- padded frames
    if (R_.fill_pad) {
        if (out_row0)
            for (int f = Tn; f < P.N; ++f) {
                float *orow = out_row0 + (size_t)f * out_ld;
                for (int k = tid; k < K; k += NT) orow[k] = -INFINITY;
            }
        if (off_seq)
            for (int f = Tn + tid; f < P.N; f += NT) off_seq[f] = 0.0;
    }
    if (R_.fmt && tid == 0) R_.fmt[b] = out_lin ? 1 : 0;   // which form this sequence's rows have
    return true;
}

template <bool LOG, int FEW, bool APART>
__global__ __launch_bounds__(kNWShared * 64) void fb_linear_kernel(const RecParams P)
{
    __builtin_amdgcn_s_setprio(3);
    extern __shared__ double lds_raw[];
    int b, which;
    if (P.started && threadIdx.x == 0) atomicAdd(P.started, 1u);   // this workgroup has its compute unit
    resolve_sequence<kNWShared>(P, lds_raw, b, which);
    if (!linear_run<false, LOG, FEW, false, APART>(P, b, which, lds_raw)) {
        recursion_run<kNWShared, float, false, kXsFixed, false>(P, b, which, lds_raw);
        if (P.dir[which].fmt && threadIdx.x == 0) P.dir[which].fmt[b] = 0;   // this sequence's rows are in the log form
    }
    count_done(P);
}

// The best path's recursions, both of them half way.  Against the back-pointer form (fb_recursion_kernel, a comparison and two selects an arc, and
// 2 bytes a state and frame instead of 4), 6000 states, 60 k arcs, 3000 pdfs, 128 sequences of 100 to 500 frames: the launch 1520 -> 870 us, the
// trace behind it 144 -> 366, a call of fb_viterbi 1606 -> 1210.  Of 7370 clocks a step the LDS is busy for 4220 (1340 of them bank conflicts) and
// a SIMD issues vector instructions in 3790, scalar ones in 1840: waves wait for half of their time, in the tail of a step above all.
template <int FEW>
__global__ __launch_bounds__(kNWShared * 64) void fb_best_linear_kernel(const RecParams P)
{
    __builtin_amdgcn_s_setprio(3);
    extern __shared__ double lds_raw[];
    int b, which;
    resolve_sequence<kNWShared>(P, lds_raw, b, which);
    linear_run<false, false, FEW, true>(P, b, which, lds_raw);
}

// The leaky-HMM's recursions (both directions, one launch); gave_up[which * B + b]: the run left its range (or the
// sequence has no frames) and is the plain kernel's.
template <int FEW>
__global__ __launch_bounds__(kNWShared * 64) void fb_leaky_linear_kernel(const RecParams P, int32_t *gave_up)
{
    __builtin_amdgcn_s_setprio(3);
    extern __shared__ double lds_raw[];
    int b, which;
    resolve_sequence<kNWShared>(P, lds_raw, b, which);
    const bool ok = linear_run<true, false, FEW>(P, b, which, lds_raw);
    if (threadIdx.x == 0) {
        gave_up[which * P.B + b] = ok ? 0 : 1;
        if (!ok) P.dir[which].fmt[b] = 1;   // (rows nobody will use, in the form the gradient kernel expects)
    }
}

template <int NW, class T, bool TROP, int XF, bool LINW = false>
__global__ __launch_bounds__(NW * 64) void fb_recursion_kernel(const RecParams P)
{
    // The large-graph kernel is the critical path of a call; small-graph launches that run beside it on the same
    // compute units (the numerators of an LF-MMI call) take the issue slots it leaves.  (The data-moving wave
    // keeps this priority; the others vary theirs within a time step.)
    if (NW == kNWShared) __builtin_amdgcn_s_setprio(3);
    extern __shared__ double lds_raw[];
    int b, which;
    if (P.started && threadIdx.x == 0) atomicAdd(P.started, 1u);   // this workgroup has its compute unit
    resolve_sequence<NW>(P, lds_raw, b, which);
    recursion_run<NW, T, TROP, XF, LINW>(P, b, which, lds_raw);
    count_done(P);
}

// ---------------------------------------------------------------------------
// Posteriors (Eq. 15) of one or two graphs and their accumulation into pdf
// posteriors; each graph enters with its sign (Eq. 17: numerator minus
// denominator).  grid = (ceil(N / frames_per_block), B), kPostThreads threads.
// A workgroup keeps the states-by-pdf tables of its sequence's graphs in LDS and
// walks its frames one at a time: log posteriors of the frame -> LDS, maximum,
// exponentials, sum, then one thread per pdf adds up the states tied to it in a
// fixed order (no atomics: results do not depend on timing).
// ---------------------------------------------------------------------------
constexpr int kPostThreads = 512;

namespace {

// First pass over one frame of one graph: log posteriors (a + b) * in_scale into stage[0..K); returns
// the thread's maximum.  IT: element type of a and b.
template <class IT>
__device__ __forceinline__ IT frame_logpost(const IT *arow, const IT *brow, IT in_scale, int K, IT *stage, int tid)
{
    IT mx = (IT)(-INFINITY);
    for (int k = tid; k < K; k += kPostThreads) {
        const IT t = (arow[k] + brow[k]) * in_scale;
        stage[k] = t;
        mx = tmax(mx, t);
    }
    return mx;
}

// Rest of the frame: block maximum, exp2(log posterior - max) into tb[0..K) (unnormalised); returns
// 1 / their sum (0 if the frame has no mass).  stage: tb itself, or a wider buffer.
template <class IT>
__device__ __forceinline__ float frame_finish(IT mx, int K, float *tb, const IT *stage, float *red, int tid, int lane, int wave)
{
    constexpr int NT = kPostThreads, NWV = kPostThreads / kWave;
    mx = wave_max(mx);
    IT *redt = (IT *)red;
    if (lane == 0) redt[wave] = mx;
    __syncthreads();
    mx = redt[0];
#pragma unroll
    for (int w = 1; w < NWV; ++w) mx = tmax(mx, redt[w]);
    __syncthreads();
    float sum = 0.0f;
    if (mx != (IT)(-INFINITY))
        for (int k = tid; k < K; k += NT) {
            const float e = fexp2((float)(stage[k] - mx));
            tb[k] = e;      // tb may alias stage when IT is float: same index, read before write
            sum += e;
        }
    else
        for (int k = tid; k < K; k += NT) tb[k] = 0.0f;
    sum = wave_sum(sum);
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    sum = red[0];
#pragma unroll
    for (int w = 1; w < NWV; ++w) sum += red[w];
    return sum > 0.0f ? 1.0f / sum : 0.0f;
}

constexpr int kPostPrefetch = 3;   // 16-byte pieces per thread and array held in registers: 6144 states

}  // namespace

__global__ __launch_bounds__(kPostThreads) void fb_posterior_kernel(const PostParams P)
{
    extern __shared__ double lds_raw[];
    constexpr int NT = kPostThreads, U = kPostPrefetch;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = P.order ? P.order[P.rank0 + blockIdx.y] : blockIdx.y;
    const int T = min(max(P.lengths[b], 0), P.N);
    const int n0 = blockIdx.x * P.frames_per_block;
    const int n_end = min(min(n0 + P.frames_per_block, P.N), T);   // real frames of this chunk: [n0, n_end)
    float *red = (float *)lds_raw;                  // reduction slots: one double or float per wave
    double *stage64 = lds_raw + 8;                  // [Kcap64] log posteriors of a double-carrier graph
    float *tb = (float *)(stage64 + P.Kcap64);      // [Kcap] per-state values of the frame
    float *rho = tb + P.Kcap;                       // [D]
    uint16_t *tab = (uint16_t *)(rho + P.D);        // per graph: row_ptr [Rcap + 1], row_pdf [Rcap], states [Kcap]
    const uint16_t *rp[2], *rd[2], *rs[2];
    PdfSub ps[2];
    // The first graph's rows of the next frame travel from HBM into registers while the current frame is
    // worked on (when it is a shared graph of float vectors whose rows are 16-byte aligned).
    const PostGraph &G0 = P.g[0];
    const int K0 = G0.pdfs.sub[0].K;
    const bool pre = G0.shared && !G0.f64 && (K0 & 3) == 0 && (G0.ld & 3) == 0 && (((uintptr_t)G0.a | (uintptr_t)G0.b) & 15) == 0 &&
                     n0 < n_end;
    const int Kpre = pre ? min(K0, NT * 4 * U) : 0;   // states covered by the prefetch registers
    float4 pa[U], pb[U];
    auto issue = [&](int n) {
        const float4 *ar = (const float4 *)((const float *)G0.a + ((size_t)b * P.N + n) * G0.ld);
        const float4 *br = (const float4 *)((const float *)G0.b + ((size_t)b * P.N + n) * G0.ld);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = u * NT + tid;
            if (q * 4 < Kpre) { pa[u] = ar[q]; pb[u] = br[q]; }
        }
    };
    if (pre) issue(n0);
    if (n0 < n_end) {   // the tables are needed only if the chunk has a real frame
        uint16_t *at = tab;
        for (int gi = 0; gi < P.n_graph; ++gi) {
            const PostGraph &G = P.g[gi];
            ps[gi] = G.pdfs.sub[G.shared ? 0 : b];
            uint16_t *p0 = at, *p1 = p0 + G.Rcap + 1, *p2 = p1 + G.Rcap;
            for (int r = tid; r <= ps[gi].n_rows; r += NT) p0[r] = G.pdfs.row_ptr[ps[gi].ptr0 + r];
            for (int r = tid; r < ps[gi].n_rows; r += NT) p1[r] = G.pdfs.row_pdf[ps[gi].row0 + r];
            for (int k = tid; k < ps[gi].K; k += NT) p2[k] = G.pdfs.states[ps[gi].st0 + k];
            rp[gi] = p0; rd[gi] = p1; rs[gi] = p2;
            at = p0 + ((2 * G.Rcap + 1 + G.Kcap + 1) & ~1);   // next table starts 4-byte aligned
        }
        __syncthreads();
    }

    for (int fi = 0; fi < P.frames_per_block; ++fi) {
        const int n = n0 + fi;
        if (n >= P.N) break;
        float *prow = P.pdf_out ? P.pdf_out + ((size_t)b * P.N + n) * P.D : nullptr;
        if (n >= T) {   // padded frame: zeros
            if (P.accumulate) continue;
            if (prow)
                for (int d = tid; d < P.D; d += NT) prow[d] = 0.0f;
            for (int gi = 0; gi < P.n_graph; ++gi) {
                const PostGraph &G = P.g[gi];
                if (!G.state_post) continue;
                const PdfSub sd = G.pdfs.sub[G.shared ? 0 : b];
                float *srow = G.shared ? G.state_post + ((size_t)b * P.N + n) * sd.K
                                       : G.state_post + (size_t)n * G.Ktot + sd.k0;
                for (int k = tid; k < sd.K; k += NT) srow[k] = 0.0f;
            }
            continue;
        }
        for (int gi = 0; gi < P.n_graph; ++gi) {
            const PostGraph &G = P.g[gi];
            const int K = ps[gi].K;
            const size_t at = G.shared ? ((size_t)b * P.N + n) * G.ld : (size_t)n * G.Ktot + ps[gi].k0;
            const bool covers_all = G.shared != 0;   // a shared graph has one row per pdf
            if (gi == 0 && !covers_all && prow && !P.accumulate)
                for (int d = tid; d < P.D; d += NT) rho[d] = 0.0f;
            float inv;
            if (G.f64) {
                const double mx = frame_logpost<double>((const double *)G.a + at, (const double *)G.b + at, (double)G.in_scale, K,
                                                        stage64, tid);
                inv = frame_finish<double>(mx, K, tb, stage64, red, tid, lane, wave);
            } else if (gi == 0 && pre) {
                float mx = -INFINITY;   // this frame's rows are in the registers
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int q = u * NT + tid;
                    if (q * 4 < Kpre) {
                        float4 t;
                        t.x = (pa[u].x + pb[u].x) * G.in_scale; t.y = (pa[u].y + pb[u].y) * G.in_scale;
                        t.z = (pa[u].z + pb[u].z) * G.in_scale; t.w = (pa[u].w + pb[u].w) * G.in_scale;
                        ((float4 *)tb)[q] = t;
                        mx = tmax(tmax(mx, tmax(t.x, t.y)), tmax(t.z, t.w));
                    }
                }
                if (n + 1 < n_end) issue(n + 1);   // the next frame starts its trip now
                if (K > Kpre)
                    mx = tmax(mx, frame_logpost<float>((const float *)G.a + at + Kpre, (const float *)G.b + at + Kpre,
                                                       G.in_scale, K - Kpre, tb + Kpre, tid));
                inv = frame_finish<float>(mx, K, tb, tb, red, tid, lane, wave);
            } else {
                const float mx = frame_logpost<float>((const float *)G.a + at, (const float *)G.b + at, G.in_scale, K, tb, tid);
                inv = frame_finish<float>(mx, K, tb, tb, red, tid, lane, wave);
            }
            if (G.state_post) {
                float *srow = G.state_post + (G.shared ? ((size_t)b * P.N + n) * K : at);
                for (int k = tid; k < K; k += NT) srow[k] = tb[k] * inv;
            }
            __syncthreads();   // tb complete (and red free again)
            if (prow) {
                const float scale = G.sign * inv;
                const uint16_t *ptr = rp[gi], *pdfid = rd[gi], *st = rs[gi];
                const int n_rows = ps[gi].n_rows;
                // tpr threads share a pdf when there are fewer pdfs than threads (tpr a power of two <= 16);
                // each thread walks two pdfs at once so that two chains of dependent LDS reads overlap
                int tpr = 1;
                while (tpr < 16 && n_rows * tpr * 2 <= NT) tpr *= 2;
                const int rpp = NT / tpr, part = tid & (tpr - 1);
                for (int r0 = tid / tpr; r0 < n_rows; r0 += 2 * rpp) {
                    const int r1 = r0 + rpp;
                    const bool two = r1 < n_rows;
                    int i0 = ptr[r0] + part, i1 = two ? ptr[r1] + part : 0;
                    const int e0 = ptr[r0 + 1], e1 = two ? ptr[r1 + 1] : 0;
                    float acc0 = 0.0f, acc1 = 0.0f;
                    while (i0 < e0 || i1 < e1) {
                        const float v0 = i0 < e0 ? tb[st[i0]] : 0.0f, v1 = i1 < e1 ? tb[st[i1]] : 0.0f;
                        acc0 += v0; acc1 += v1;
                        i0 += tpr; i1 += tpr;
                    }
                    for (int o = tpr >> 1; o >= 1; o >>= 1) {   // fixed order: results do not depend on timing
                        acc0 += __shfl_xor(acc0, o, 64);
                        acc1 += __shfl_xor(acc1, o, 64);
                    }
                    if (part == 0) {
                        if (P.accumulate) {   // straight into the caller's row: a sequence's rows name distinct pdfs
                            prow[pdfid[r0]] += acc0 * scale;
                            if (two) prow[pdfid[r1]] += acc1 * scale;
                        } else {
                            if (gi == 0 && covers_all) rho[pdfid[r0]] = acc0 * scale;
                            else rho[pdfid[r0]] += acc0 * scale;
                            if (two) {
                                if (gi == 0 && covers_all) rho[pdfid[r1]] = acc1 * scale;
                                else rho[pdfid[r1]] += acc1 * scale;
                            }
                        }
                    }
                }
                __syncthreads();
            }
        }
        if (prow && !P.accumulate)
            for (int d = tid; d < P.D; d += NT) prow[d] = rho[d];
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Gradient of the LF-MMI objective (Eq. 17) for the usual pair of graphs: a shared
// denominator whose vectors are float, packed numerators with at most kGradNumK
// states and pdf rows each (or the denominator's share alone), for calls whose
// recursions also left the running sums of their offsets (PostParams::cum_a, cum_b:
// A_n, B_n with alpha_n = stored row + A_n, beta_n = stored row + B_n, log2 units)
// and log Z.  Same sums in the same order as fb_posterior_kernel, organised for speed:
// grid = (ceil(N / frames_per_block), B), 8 waves, one workgroup barrier per frame.  (Eight, two per SIMD: two
// workgroups then share a compute unit.  With nine - three on one SIMD - the second workgroup was never placed
// beside the first, whatever the occupancy calculation says, and the kernel ran at 3/4 of its present rate.)
// Waves 0-6 work on the denominator: a thread keeps, for the whole block, the
// places of "its" states in pdf order and the state ranges of "its" pdfs in
// registers, the rows of the next frame travel from HBM into registers while the
// current frame is worked on, and the exponentials go to LDS in pdf order, so that a
// pdf's states are neighbours.  The exponentials of a frame are taken of
//   t_k - (log2 Z - A_n - B_n) = log2 of the posterior itself (<= 0, largest >= -log2 K),
// so no maximum over the frame, no reduction of it over the workgroup and no barrier
// behind it are needed (the values are still normalised by their own sum, so a drift
// of the float recursions cancels).  The denominator waves store their pdf posteriors
// straight from the sums (no staging of the row in LDS), adding the numerator's value
// for the pdf, which wave 7 - it works on the numerator of the same frame at the same
// time, with wave-level reductions only - has left in a small list (two buffers, by
// frame parity) before the frame's barrier; the exponentials in pdf order have two
// buffers as well, so nothing of frame n + 1 overwrites what frame n still reads.
// Without the offsets (the pdf posteriors of fb_posteriors: one shared graph, rows of logarithms as fb_alpha and
// fb_beta return them) the frame's largest sum of a forward and a backward entry takes the place of
// log2 Z - A_n - B_n: one more reduction over the workgroup and a second barrier per frame.
// LDS: red [2][16] sums and [2][16] maxima of waves 0-6; tb [2][K0 rounded to 4, + kGradSlack]; nval [2][Rcap] the numerator's pdf
// posteriors by pdf row; en [Kcap] numerator exponentials; nidx [D] 16-bit: pdf -> its row in
// this sequence's numerator + 1, 0 = none; the numerator tables.
// ---------------------------------------------------------------------------
constexpr int kGradMain = 448, kGradThreads = kGradMain + kWave;
constexpr int kGradU = 4;        // 16-byte pieces of a denominator row per thread: 7168 states
constexpr int kGradPdf = 8;      // pdfs per thread: 3584 pdfs
constexpr int kGradNumU = 8;     // numerator states (and pdf rows) per lane: 512
constexpr int kGradNumK = kGradNumU * kWave;
constexpr int kGradAhead = 8;    // states of a pdf whose exponentials are read at once, before any of them is added
constexpr int kGradSlack = 4 + kGradAhead;   // floats behind a buffer of exponentials: reads ahead may pass the last state

// a 16-byte load of data that is read once: it should not push the recursion kernel's arc plan out of L2
__device__ __forceinline__ float4 nt_load4(const float4 *p)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 v = __builtin_nontemporal_load((const f4 *)p);
    return make_float4(v.x, v.y, v.z, v.w);
}

// four consecutive floats of a row whose pieces need not be 16-byte aligned; have: how many of them exist (the
// others come back as 0 and nothing behind the row is touched)
__device__ __forceinline__ float4 nt_load4_any(const float *p, int have)
{
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
    if (have >= 4) {
        const f4u v = __builtin_nontemporal_load((const f4u *)p);
        return make_float4(v.x, v.y, v.z, v.w);
    }
    float4 r = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (have > 0) r.x = p[0];
    if (have > 1) r.y = p[1];
    if (have > 2) r.z = p[2];
    return r;
}

template <class NT>
__global__ __launch_bounds__(kGradThreads, 4) void fb_grad_kernel(const PostParams P)
{
    extern __shared__ double lds_raw[];
    constexpr int MT = kGradMain, U = kGradU, NU = kGradNumU;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool den_side = wave < MT / kWave;
    const int b = P.order ? P.order[P.rank0 + blockIdx.y] : blockIdx.y;
    const int T = min(max(P.lengths[b], 0), P.N);
    const int n0 = blockIdx.x * P.frames_per_block;
    const int n_end = min(min(n0 + P.frames_per_block, P.N), T);   // real frames of this chunk: [n0, n_end)
    // one graph, or a second graph whose vectors were not complete when the launch was released (PostParams::fused):
    // the shared graph's share alone (no numerators: wave 7 only keeps the barriers)
    const bool has_num = P.n_graph == 2 && (!P.fused || *P.fused != 0);
    const PostGraph &G0 = P.g[0], &G1 = P.g[1];
    const int K0 = G0.pdfs.sub[0].K, D = P.D;
    const int K0r = ((K0 + 3) & ~3) + kGradSlack;
    const PdfSub ps1 = has_num ? G1.pdfs.sub[b] : PdfSub{};
    const int K1 = ps1.K, R1 = ps1.n_rows;

    float *red = (float *)lds_raw;                       // [2][16] sums, [2][16] maxima
    float *tb = red + 64;                                // [2][K0r]
    float *nval = tb + 2 * K0r;                          // [2][Rcap]
    float *en = nval + 2 * G1.Rcap;                      // [Kcap]
    uint16_t *nidx = (uint16_t *)(en + G1.Kcap);         // [D rounded to 2]
    uint16_t *nptr = nidx + ((D + 1) & ~1);              // numerator tables: row_ptr [Rcap + 1], row_pdf [Rcap], states [Kcap]
    uint16_t *npdf = nptr + G1.Rcap + 1, *nst = npdf + G1.Rcap;

    for (int n = n0 + (n_end > n0 ? n_end - n0 : 0); n < min(n0 + P.frames_per_block, P.N); ++n) {   // padded frames: zeros
        float *prow = P.pdf_out + ((size_t)b * P.N + n) * D;
        for (int d = tid; d < D; d += kGradThreads) prow[d] = 0.0f;
    }
    if (n0 >= n_end) return;

    // which numerator row a pdf has (the same for every frame of the block)
    for (int d = tid; d < D; d += kGradThreads) nidx[d] = 0;
    __syncthreads();
    for (int r = tid; r < R1; r += kGradThreads) nidx[G1.pdfs.row_pdf[ps1.row0 + r]] = (uint16_t)(r + 1);   // (R1 = 0 without numerators)
    // (visible to the denominator waves after the first frame's barrier)

    if (den_side) {
        float4 pa[U], pb[U];          // rows of the frame being prefetched / worked on
        float ca, cb;                 // A_n, B_n of that frame
        uint2 posr[U];                // places (4 x 16 bit) of the thread's states in pdf order
        uint32_t prange[kGradPdf];    // state ranges (begin | end << 16) of the thread's pdfs tid, tid + MT, ...
        const double z2 = P.logz ? P.logz[b] * kLog2e : 0.0;   // log2 Z of the shared graph
        // rows in whole 16-byte pieces (the workspace of an LF-MMI call; the caller's rows when K is a multiple of 4)
        const bool pieces16 = (G0.ld & 3) == 0 && (((uintptr_t)G0.a | (uintptr_t)G0.b) & 15) == 0;
        const bool by_max = !P.cum_a;   // no offsets: the frame's exponentials are taken relative to its largest sum
        // the form of this sequence's rows: the values themselves (what the probability-domain recursion leaves), or logs
        const bool lin_a = G0.fmt_a && G0.fmt_a[b] != 0, lin_b = G0.fmt_b && G0.fmt_b[b] != 0;
        const bool any_lin = lin_a || lin_b;
        const float in_scale0 = G0.in_scale;
        auto as_value = [in_scale0](float v, bool lin) -> double {   // a row entry as a double: itself, or 2^(its log2)
            if (lin) return (double)v;
            const float x = v * in_scale0;
            if (!(x > -1.0e30f)) return 0.0;
            const float fl = floorf(x);
            return ldexp((double)fexp2(x - fl), (int)fl);
        };
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = u * MT + tid;
            posr[u] = q * 4 < K0 ? ((const uint2 *)G0.pdfs.pos)[q] : make_uint2(0u, 0u);
        }
        // Few pdfs (the paper's own graphs: 84 pdfs for 3022 states): tpp threads, neighbours in a wave, share a pdf,
        // each with a part of its states; their sums are added in a fixed order.  Otherwise a thread has up to
        // kGradPdf whole pdfs: tid, tid + MT, ...
        int tpp = 1;
        while (tpp < kWave && D * tpp * 2 <= MT) tpp *= 2;
        const int n_mine = tpp > 1 ? 1 : kGradPdf;   // pdfs (or parts of one) of a thread
#pragma unroll
        for (int j = 0; j < kGradPdf; ++j) {
            const int d = tpp > 1 ? tid / tpp : j * MT + tid;
            uint32_t lo = 0, hi = 0;
            if (d < D && j < n_mine) {
                lo = G0.pdfs.row_ptr[d];
                hi = G0.pdfs.row_ptr[d + 1];
                if (tpp > 1) {
                    const uint32_t len = hi - lo, part = (uint32_t)(tid & (tpp - 1));
                    hi = lo + len * (part + 1) / (uint32_t)tpp;
                    lo = lo + len * part / (uint32_t)tpp;
                }
            }
            prange[j] = lo | (hi << 16);
        }
        // the most states any pdf of this wave has: how far the reads ahead below go is the same for all its lanes
        float most = 0.0f;
#pragma unroll
        for (int j = 0; j < kGradPdf; ++j) most = tmax(most, (float)((prange[j] >> 16) - (prange[j] & 0xffffu)));
        const int wcnt = __builtin_amdgcn_readfirstlane((int)wave_max(most));
        // The frames of the block, for one form of the rows: 2 both hold values (every sequence the probability-domain
        // recursion has carried through), 0 both hold logs, 1 one of each (a sequence that fell back in one direction).
        auto frames = [&](auto form_c, auto few_c) {
        constexpr int form = decltype(form_c)::value;
        constexpr bool few = decltype(few_c)::value;   // few pdfs: several threads share one (tpp > 1)
        auto issue = [&](int n) {
            const float *af = (const float *)G0.a + ((size_t)b * P.N + n) * G0.ld;
            const float *bf = (const float *)G0.b + ((size_t)b * P.N + n) * G0.ld;
            const float4 *ar = (const float4 *)af, *br = (const float4 *)bf;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = u * MT + tid;
                if (q * 4 < K0) {
                    // (rows that hold values are the workspace's: whole pieces)
                    if (form != 0 || pieces16) { pa[u] = nt_load4(ar + q); pb[u] = nt_load4(br + q); }
                    else { pa[u] = nt_load4_any(af + q * 4, K0 - q * 4); pb[u] = nt_load4_any(bf + q * 4, K0 - q * 4); }
                }
            }
            ca = (form == 0 && by_max) ? 0.0f : P.cum_a[(size_t)b * P.N + n];   // (rows that hold values come with offsets)
            cb = (form == 0 && by_max) ? 0.0f : P.cum_b[(size_t)b * P.N + n];
        };
        issue(n0);
        for (int n = n0; n < n_end; ++n) {
            const int par = (n - n0) & 1;
            float *tbn = tb + par * K0r;
            // (the packed places and ranges stay packed between frames: unpacked once and for all they would not fit
            // the registers)
#pragma unroll
            for (int u = 0; u < U; ++u) asm volatile("" : "+v"(posr[u].x), "+v"(posr[u].y));
#pragma unroll
            for (int j = 0; j < kGradPdf; ++j) asm volatile("" : "+v"(prange[j]));
            // log2 Z - A_n - B_n; a sequence without any path (log Z = -inf) has no posteriors
            double shift_d = z2 - (double)ca - (double)cb;
            if (form == 0 && by_max) {
                // Rows without offsets (normalised logs as fb_alpha / fb_beta return them): the largest sum of the
                // frame takes the place of log2 Z - A_n - B_n, at the price of a second barrier per frame.
                float mx = -INFINITY;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int q = u * MT + tid;
                    if (q * 4 < K0) {
                        mx = tmax(mx, pa[u].x + pb[u].x);
                        if (q * 4 + 1 < K0) mx = tmax(mx, pa[u].y + pb[u].y);
                        if (q * 4 + 2 < K0) mx = tmax(mx, pa[u].z + pb[u].z);
                        if (q * 4 + 3 < K0) mx = tmax(mx, pa[u].w + pb[u].w);
                    }
                }
                mx = wave_max(mx);
                if (lane == 0) red[32 + par * 16 + wave] = mx;
                __syncthreads();
                mx = red[32 + par * 16];
#pragma unroll
                for (int w = 1; w < MT / kWave; ++w) mx = tmax(mx, red[32 + par * 16 + w]);
                shift_d = mx > -INFINITY ? (double)(mx * G0.in_scale) : -INFINITY;
            }
            const bool mass = shift_d > -1.0e300 && shift_d < 1.0e300;
            const float shift = mass ? (float)shift_d : 0.0f;
            // 2^-shift in double, for rows that hold values instead of logs (their range is a float's, times the offsets')
            double pow_shift = 0.0;
            if (form != 0 && mass) {
                const double t = fmin(fmax(-shift_d, -2000.0), 2000.0), ti = floor(t);
                pow_shift = ldexp((double)fexp2((float)(t - ti)), (int)ti);
            }
            float sum = 0.0f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = u * MT + tid;
                if (q * 4 < K0) {
                    float e[4];
                    if (form == 2) {   // rows that hold the values themselves: the posterior is their product, formed in double
                        e[0] = (float)((double)pa[u].x * (double)pb[u].x * pow_shift);
                        e[1] = (float)((double)pa[u].y * (double)pb[u].y * pow_shift);
                        e[2] = (float)((double)pa[u].z * (double)pb[u].z * pow_shift);
                        e[3] = (float)((double)pa[u].w * (double)pb[u].w * pow_shift);
                    } else if (form == 1) {
                        e[0] = (float)(as_value(pa[u].x, lin_a) * as_value(pb[u].x, lin_b) * pow_shift);
                        e[1] = (float)(as_value(pa[u].y, lin_a) * as_value(pb[u].y, lin_b) * pow_shift);
                        e[2] = (float)(as_value(pa[u].z, lin_a) * as_value(pb[u].z, lin_b) * pow_shift);
                        e[3] = (float)(as_value(pa[u].w, lin_a) * as_value(pb[u].w, lin_b) * pow_shift);
                    } else {
                        e[0] = fexp2((pa[u].x + pb[u].x) * G0.in_scale - shift); e[1] = fexp2((pa[u].y + pb[u].y) * G0.in_scale - shift);
                        e[2] = fexp2((pa[u].z + pb[u].z) * G0.in_scale - shift); e[3] = fexp2((pa[u].w + pb[u].w) * G0.in_scale - shift);
                    }
                    if (q * 4 + 3 >= K0) {   // the row's last piece when K0 is not a multiple of 4: padding counts as zero-bar
                        if (q * 4 + 1 >= K0) e[1] = 0.0f;
                        if (q * 4 + 2 >= K0) e[2] = 0.0f;
                        e[3] = 0.0f;
                    }
                    if (!mass) e[0] = e[1] = e[2] = e[3] = 0.0f;
                    sum += (e[0] + e[1]) + (e[2] + e[3]);
                    tbn[posr[u].x & 0xffffu] = e[0]; tbn[posr[u].x >> 16] = e[1];
                    tbn[posr[u].y & 0xffffu] = e[2]; tbn[posr[u].y >> 16] = e[3];
                }
                __builtin_amdgcn_sched_barrier(0);   // one piece at a time: the doubles of all at once would not fit the registers
            }
            if (n + 1 < n_end) issue(n + 1);   // the next frame starts its trip now
            sum = wave_sum(sum);
            if (lane == 0) red[par * 16 + wave] = sum;
            __syncthreads();                       // the frame's only barrier
            sum = red[par * 16];
#pragma unroll
            for (int w = 1; w < MT / kWave; ++w) sum += red[par * 16 + w];
            const float scale = sum > 0.0f ? G0.sign / sum : 0.0f;
            float *prow = P.pdf_out + ((size_t)b * P.N + n) * D;
            const float *nv = nval + par * G1.Rcap;
            // A pdf's exponentials are neighbours in the buffer.  The first kGradAhead of each of two pdfs are read
            // at once (as far as the wave's longest pdf goes; what lies behind a pdf's own states is read and not
            // used), so that a thread waits for LDS once per two pdfs and not once per state; they are added in
            // ascending order of states as before, and what a pdf has beyond them in a loop of its own.
            constexpr int H = 2;
            static_assert(kGradPdf % H == 0, "pdfs per thread come in groups");
#pragma unroll
            for (int h = 0; h < (few ? 1 : kGradPdf); h += H) {
                float t[H][kGradAhead];
                uint32_t r[H];
#pragma unroll
                for (int jj = 0; jj < H; ++jj) {
                    const float *seg = tbn + (prange[h + jj] & 0xffffu);
#pragma unroll
                    for (int i = 0; i < kGradAhead; i += 2)
                        if (wcnt > i) { t[jj][i] = seg[i]; t[jj][i + 1] = seg[i + 1]; }
                    r[jj] = nidx[min(few ? tid / tpp : (h + jj) * MT + tid, D - 1)];
                }
                float nvv[H];
#pragma unroll
                for (int jj = 0; jj < H; ++jj) nvv[jj] = nv[r[jj] ? r[jj] - 1 : 0];   // (no numerators: never used)
#pragma unroll
                for (int jj = 0; jj < H; ++jj) {
                    const int d = few ? tid / tpp : (h + jj) * MT + tid;
                    const int begin = (int)(prange[h + jj] & 0xffffu), end = (int)(prange[h + jj] >> 16);
                    float acc = 0.0f;
#pragma unroll
                    for (int i = 0; i < kGradAhead; ++i)
                        if (wcnt > i) acc += begin + i < end ? t[jj][i] : 0.0f;
                    if (wcnt > kGradAhead)
                        for (int i = begin + kGradAhead; i < end; ++i) acc += tbn[i];
                    if (few)
                        for (int o = 1; o < tpp; o <<= 1) acc += __shfl_xor(acc, o, kWave);   // the parts of a pdf, in a fixed order
                    // (a product and a sum, each rounded: the bits a launch of the denominator's share followed by one
                    // that adds the numerators' gives, whichever of the two ways a call takes)
                    float v = acc * scale;
                    asm volatile("" : "+v"(v));   // (kept a product of its own: not merged with the sum into one rounding)
                    if (r[jj]) v += nvv[jj];
                    if (few ? (d < D && (tid & (tpp - 1)) == 0 && jj == 0) : d < D) __builtin_nontemporal_store(v, prow + d);
                }
            }
        }
        };
        const std::true_type yes;
        const std::false_type no;
        if (tpp > 1) {
            if (lin_a && lin_b) frames(std::integral_constant<int, 2>(), yes);
            else if (any_lin) frames(std::integral_constant<int, 1>(), yes);
            else frames(std::integral_constant<int, 0>(), yes);
        } else {
            if (lin_a && lin_b) frames(std::integral_constant<int, 2>(), no);
            else if (any_lin) frames(std::integral_constant<int, 1>(), no);
            else frames(std::integral_constant<int, 0>(), no);
        }
    } else {
        NT qa[NU], qb[NU];            // rows of the frame being prefetched / worked on
        auto issue = [&](int n) {
            const NT *ar = (const NT *)G1.a + (size_t)n * G1.Ktot + ps1.k0, *br = (const NT *)G1.b + (size_t)n * G1.Ktot + ps1.k0;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int k = u * kWave + lane;
                if (k < K1) { qa[u] = ar[k]; qb[u] = br[k]; }
            }
        };
        if (!has_num) {
            const bool two = !P.cum_a && !(G0.fmt_a && G0.fmt_a[b] != 0) && !(G0.fmt_b && G0.fmt_b[b] != 0);   // as the other waves decide
            for (int n = n0; n < n_end; ++n) {
                if (two) __syncthreads();
                __syncthreads();
            }
            return;
        }
        issue(n0);
        for (int r = lane; r <= R1; r += kWave) nptr[r] = G1.pdfs.row_ptr[ps1.ptr0 + r];
        for (int k = lane; k < K1; k += kWave) nst[k] = G1.pdfs.states[ps1.st0 + k];
        for (int n = n0; n < n_end; ++n) {
            const int par = (n - n0) & 1;
            NT t[NU];
            NT mx = (NT)(-INFINITY);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int k = u * kWave + lane;
                if (k < K1) {
                    t[u] = (qa[u] + qb[u]) * (NT)G1.in_scale;
                    mx = tmax(mx, t[u]);
                }
            }
            if (n + 1 < n_end) issue(n + 1);
            mx = wave_max(mx);
            float sum = 0.0f;
            const bool mass = mx != (NT)(-INFINITY);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the previous frame's reads of en come first
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int k = u * kWave + lane;
                if (k < K1) {
                    const float e = mass ? fexp2((float)(t[u] - mx)) : 0.0f;
                    en[k] = e;
                    sum += e;
                }
            }
            sum = wave_sum(sum);
            const float scale = sum > 0.0f ? G1.sign / sum : 0.0f;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wave's writes of en (and of its tables) before its reads
            float *nv = nval + par * G1.Rcap;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int r = u * kWave + lane;
                if (r < R1) {
                    float acc = 0.0f;
                    for (int i = nptr[r]; i < nptr[r + 1]; ++i) acc += en[nst[i]];
                    nv[r] = acc * scale;
                }
            }
            __syncthreads();                       // the frame's only barrier: the denominator waves may read nv
        }
    }
}

// The pdf posteriors of small packed graphs (at most kGradNumK states and pdf rows each; the numerators of an
// LF-MMI call) added, with the graph's sign, to rows that already hold another graph's share (PostParams::accumulate).
// grid = (ceil(N / frames_per_block), B), one wave per workgroup: the wave walks its frames as the last wave of
// fb_grad_kernel does (same arithmetic, same order), with the rows of the next frame on their way while it works,
// and adds straight into the caller's rows: a sequence's pdf rows name distinct pdfs, padded frames are left alone.
template <class NT>
__global__ __launch_bounds__(kWave) void fb_num_add_kernel(const PostParams P)
{
    extern __shared__ double lds_raw[];
    constexpr int NU = kGradNumU;
    const int lane = threadIdx.x;
    const int b = P.order ? P.order[P.rank0 + blockIdx.y] : blockIdx.y;
    const int T = min(max(P.lengths[b], 0), P.N);
    const int n0 = blockIdx.x * P.frames_per_block;
    const int n_end = min(n0 + P.frames_per_block, T);   // real frames of this chunk: [n0, n_end)
    if (n0 >= n_end) return;
    if (P.fused && *P.fused != 0) return;   // the launch before this one has added this graph's share already
    const PostGraph &G1 = P.g[0];
    const PdfSub ps1 = G1.pdfs.sub[b];
    const int K1 = ps1.K, R1 = ps1.n_rows;
    float *en = (float *)lds_raw;                        // [Kcap] exp(log posterior - max)
    uint16_t *nptr = (uint16_t *)(en + G1.Kcap);         // row_ptr [Rcap + 1], row_pdf [Rcap], states [Kcap]
    uint16_t *npdf = nptr + G1.Rcap + 1, *nst = npdf + G1.Rcap;
    NT qa[NU], qb[NU];
    auto issue = [&](int n) {
        const NT *ar = (const NT *)G1.a + (size_t)n * G1.Ktot + ps1.k0, *br = (const NT *)G1.b + (size_t)n * G1.Ktot + ps1.k0;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int k = u * kWave + lane;
            if (k < K1) { qa[u] = ar[k]; qb[u] = br[k]; }
        }
    };
    issue(n0);
    for (int r = lane; r <= R1; r += kWave) nptr[r] = G1.pdfs.row_ptr[ps1.ptr0 + r];
    for (int r = lane; r < R1; r += kWave) npdf[r] = G1.pdfs.row_pdf[ps1.row0 + r];
    for (int k = lane; k < K1; k += kWave) nst[k] = G1.pdfs.states[ps1.st0 + k];
    for (int n = n0; n < n_end; ++n) {
        NT t[NU];
        NT mx = (NT)(-INFINITY);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int k = u * kWave + lane;
            if (k < K1) {
                t[u] = (qa[u] + qb[u]) * (NT)G1.in_scale;
                mx = tmax(mx, t[u]);
            }
        }
        if (n + 1 < n_end) issue(n + 1);
        mx = wave_max(mx);
        float sum = 0.0f;
        const bool mass = mx != (NT)(-INFINITY);
        __syncthreads();   // (one wave: orders the previous frame's reads of en before these writes)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int k = u * kWave + lane;
            if (k < K1) {
                const float e = mass ? fexp2((float)(t[u] - mx)) : 0.0f;
                en[k] = e;
                sum += e;
            }
        }
        sum = wave_sum(sum);
        const float scale = sum > 0.0f ? G1.sign / sum : 0.0f;
        __syncthreads();   // the writes of en (and, in the first frame, of the tables) before the reads below
        float *prow = P.pdf_out + ((size_t)b * P.N + n) * P.D;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int r = u * kWave + lane;
            if (r < R1) {
                float acc = 0.0f;
                for (int i = nptr[r]; i < nptr[r + 1]; ++i) acc += en[nst[i]];
                float share = acc * scale;
                asm volatile("" : "+v"(share));   // (rounded as the gradient kernel's last wave rounds it, then added)
                prow[npdf[r]] += share;
            }
        }
    }
}

// order[rank] = b: the sequences by length, longest first (equal lengths by index).  One thread per sequence
// counts the sequences that go before its own.
__global__ __launch_bounds__(256) void fb_order_kernel(const int32_t *lengths, int32_t B, int32_t N, int32_t *order, uint32_t *done)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (done && b <= kDoneStarted) done[b] = 0u;   // the progress counters of the call start at zero
    if (b >= B) return;
    const int lb = min(max(lengths[b], 0), N);
    int rank = 0;
    for (int j = 0; j < B; ++j) {
        const int lj = min(max(lengths[j], 0), N);
        rank += (lj > lb || (lj == lb && j < b)) ? 1 : 0;
    }
    order[rank] = b;
}

// loss = sum_b (log Z_num[b] - log Z_den[b]) over the sequences that have frames (Eq. 16),
// summed in double in a fixed order.
__global__ __launch_bounds__(256) void fb_loss_kernel(const double *zn, const double *zd, const int32_t *lengths, int32_t B,
                                                      double *loss)
{
    __shared__ double acc[256];
    double a = 0.0;
    for (int b = threadIdx.x; b < B; b += 256)
        if (lengths[b] > 0) a += zn[b] - zd[b];
    acc[threadIdx.x] = a;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if ((int)threadIdx.x < s) acc[threadIdx.x] += acc[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = acc[0];
}

// Best path: the two halves joined and followed.  The recursions have left, at the frame m where they met (path_middle),
// the best score from the start to every state there and from every state there to the end; their largest sum is the
// score, the state that attains it the path's at frame m (of equal ones the smallest), and the back-pointers lead from
// there to both ends.  One workgroup per sequence and half.
// A path is a chain of dependent reads (the back-pointer of a frame names the row entry to read at the next one), each
// a trip to HBM if taken one by one; so the workgroup copies the sequence's back-pointer rows of several frames at a
// time into LDS (whole rows: which entry is needed is only known once the chain gets there), the next block travelling
// while one thread walks the frames of this one there.  That thread's wave asks for nothing and stores nothing: a wait
// for an LDS read is also one for every load and store its wave has on the way (the copies write LDS), and a store per
// frame made a step of the walk 0.3 us.  Whole calls of fb_viterbi, before and after: 32 label-sequence graphs over 209
// frames 70.7 -> 53.4 us; 6000 states, 128 sequences of at most 500 frames 1670 -> 1644 us (with 3 instead of 7 copying
// waves 1681).  Bound: reading the rows once (466 MB for 128 sequences of at
// most 500 frames over 6000 states: 250 us as one chain per sequence, on half as many compute units; 161 us as two).
// Indices are those of the state buffers (a state, or Kcap + slot for a clone of a very long row, which each direction
// has for itself); a clone is reported as the state it belongs to.
constexpr int kBtThreads = 512, kBtFrames = 64;
constexpr size_t kBtSmallBytes = 64 * 1024;   // rows in LDS beyond this only as far as kBtLargeFrames
constexpr int kBtLargeFrames = 8;
static_assert(kBtFrames <= kWave, "a lane hands over a frame");

__global__ __launch_bounds__(kBtThreads) void fb_backtrace_kernel(const BacktraceParams P)
{
    extern __shared__ uint16_t bt_rows[];   // [2][frames][W]: the 16-byte pieces that hold the states' columns, then the clone slots'
    const int b = blockIdx.x % P.B, half = blockIdx.x / P.B, tid = threadIdx.x;   // half 0: frames m .. 0, 1: m + 1 .. T - 1
    auto sub_of = [&](int h) {
        SubDesc sd{};
        if (P.small_sub) {
            sd.k0 = P.small_sub[P.shared ? 0 : b].k0;
            sd.K = P.small_sub[P.shared ? 0 : b].K;
        } else {
            sd = P.sched[h].sub[P.shared ? 0 : b];
        }
        return sd;
    };
    const SubDesc sd0 = sub_of(0), sd1 = sub_of(1);
    const CloneDesc *const cd0 = P.sched[0].clones + sd0.clone0, *const cd1 = P.sched[1].clones + sd1.clone0;
    const int n_cd0 = sd0.n_cdesc, n_cd1 = sd1.n_cdesc;
    const int T = min(max(P.lengths[b], 0), P.N), m = path_middle(T);
    const int k0 = sd0.k0, K = sd0.K, F = P.frames;
    int32_t *prow = P.path + (size_t)b * P.N;
    if (half == 0)
        for (int n = T + tid; n < P.N; n += kBtThreads) prow[n] = -1;
    if (T == 0) {
        if (half == 0 && tid == 0) P.score[b] = -INFINITY;
        return;
    }
    // where the sequence's columns lie in a row of back-pointers, and the 16-byte pieces of the row that hold them
    // (rows are a multiple of 8 entries long and start on 16-byte boundaries)
    const int64_t col_states = P.shared ? 0 : k0;
    const int64_t col_clones = P.shared ? (int64_t)K : (int64_t)P.Ktot + (int64_t)b * P.Ccap;
    const int64_t ps0 = col_states >> 3, ps1 = (col_states + K + 7) >> 3;
    const int64_t pc0 = col_clones >> 3, pc1 = (col_clones + P.Ccap + 7) >> 3;
    const int ns = (int)(ps1 - ps0), nc = P.Ccap > 0 ? (int)(pc1 - pc0) : 0;   // pieces
    const int W = (ns + nc) * 8;
    const int at_states = (int)(col_states - ps0 * 8), at_clones = ns * 8 + (int)(col_clones - pc0 * 8);
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the half's rows in the order it takes them: m, m - 1, .. 1 or m + 1, .. T - 1; in blocks of F, in two buffers: the
    // next block is on its way from global memory while thread 0 walks this one
    const int n_rows = half ? T - 1 - m : m;
    auto row_of = [&](int i) { return half ? m + 1 + i : m - i; };
    // rows row_of(i0), ..., straight into LDS, 16 bytes per lane, nothing waits in between; by all waves but the first, a
    // wave's worth of pieces of a row each in turn
    auto issue = [&](int i0, int buf) {
        if (wave == 0) return;
        const int cnt = min(F, n_rows - i0);
        auto span = [&](int64_t piece0, int n, int to) {
            const int nr = (n + kWave - 1) & ~(kWave - 1);
            if (nr == 0) return;
            for (int f = 0, p = (wave - 1) * kWave; ; p += kBtThreads - kWave) {
                while (p >= nr) { p -= nr; ++f; }
                if (f >= cnt) break;
                const uint4 *row = (const uint4 *)(P.bp + (P.shared ? ((size_t)b * P.N + row_of(i0 + f)) : (size_t)row_of(i0 + f)) * P.bp_ld);
                uint4 *dst = (uint4 *)(bt_rows + ((size_t)buf * F + f) * W) + to;
                if (p + lane < n)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + piece0 + p + lane),
                                                     (__attribute__((address_space(3))) void *)(dst + p), 16, 0, 0);
            }
        };
        span(ps0, ns, 0);
        span(pc0, nc, ns);
    };
    if (n_rows > 0) issue(0, 0);

    // ---- the score and the places of its path in both directions' vectors (both workgroups of a sequence find the same)
    const size_t mid_at = (size_t)b * P.mid_ld;
    auto value = [&](int h, int idx) {
        return P.f64 ? ((const double *)P.mid[h])[mid_at + idx] : (double)((const float *)P.mid[h])[mid_at + idx];
    };
    auto value1 = [&](int idx) { return value(1, idx); };
    double best = -INFINITY;
    uint32_t at = 0xffffffffu;   // place in the forward vector << 16 | place in the backward vector
    auto take = [&](double v, uint32_t a) {
        if (v > best || (v == best && a < at)) { best = v; at = a; }
    };
    for (int k = tid; k < K; k += kBtThreads) {
        const double v = value(0, k) + value1(k);
        if (v > best) { best = v; at = (uint32_t)k << 16 | (uint32_t)k; }   // (a lane's states come in ascending order)
    }
    // a cloned state's value is the largest of its own and its clones'; a clone's way on starts where its state's does
    for (int j = tid; j < n_cd0; j += kBtThreads) {
        const CloneDesc c = cd0[j];
        for (int i = 0; i < c.count; ++i) {
            const uint32_t f = (uint32_t)(P.Kcap + c.first + i);
            const double v = value(0, (int)f);
            take(v + value1(c.state), f << 16 | (uint32_t)c.state);
            for (int j1 = 0; j1 < n_cd1; ++j1)
                if (cd1[j1].state == c.state)
                    for (int i1 = 0; i1 < cd1[j1].count; ++i1) {
                        const uint32_t f1 = (uint32_t)(P.Kcap + cd1[j1].first + i1);
                        take(v + value1((int)f1), f << 16 | f1);
                    }
        }
    }
    for (int j = tid; j < n_cd1; j += kBtThreads) {
        const CloneDesc c = cd1[j];
        const double v = value(0, c.state);
        for (int i = 0; i < c.count; ++i) {
            const uint32_t f1 = (uint32_t)(P.Kcap + c.first + i);
            take(v + value1((int)f1), (uint32_t)c.state << 16 | f1);
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const double v = __shfl_xor(best, o, 64);
        const uint32_t a = (uint32_t)__shfl_xor((int)at, o, 64);
        take(v, a);
    }
    double *red_v = (double *)(bt_rows + (size_t)2 * F * W);   // [waves] the waves' best, [waves] their places
    uint32_t *red_a = (uint32_t *)(red_v + kBtThreads / kWave);
    uint16_t *const walked = (uint16_t *)(red_a + kBtThreads / kWave);   // [2][kBtFrames] what thread 0 has found in a block
    if (lane == 0) { red_v[wave] = best; red_a[wave] = at; }
    __syncthreads();
    best = red_v[0]; at = red_a[0];
#pragma unroll
    for (int w = 1; w < kBtThreads / kWave; ++w) take(red_v[w], red_a[w]);
    const bool none = best == -INFINITY;
    if (half == 0 && tid == 0)
        P.score[b] = none ? -INFINITY : (P.mid_off[0][b] + P.mid_off[1][b] + best) * kLn2;
    if (none) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (rows on their way into this workgroup's LDS)
        for (int i = tid; i < (half ? n_rows : m + 1); i += kBtThreads) prow[half ? m + 1 + i : i] = -1;
        return;
    }

    // ---- along the back-pointers
    const CloneDesc *const cdesc = half ? cd1 : cd0;
    const int n_cdesc = half ? n_cd1 : n_cd0;
    auto state_of = [&](int idx) {
        if (idx < P.Kcap) return idx;
        const int slot = idx - P.Kcap;
        int state = 0;
        for (int j = 0; j < n_cdesc; ++j)
            if (slot >= cdesc[j].first && slot < cdesc[j].first + cdesc[j].count) state = cdesc[j].state;
        return state;
    };
    int s = half ? (int)(at & 0xffffu) : (int)(at >> 16);
    if (half == 0 && tid == 0) prow[m] = k0 + state_of(s);
    // thread 0 keeps what it finds in LDS and a lane each of the second wave hands it over once the block is done
    auto hand_over = [&](int i0, int buf) {
        if (wave == 1 && lane < min(F, n_rows - i0))
            prow[half ? row_of(i0 + lane) : row_of(i0 + lane) - 1] = k0 + state_of(walked[buf * kBtFrames + lane]);
    };
    for (int i0 = 0, buf = 0; i0 < n_rows; i0 += F, buf ^= 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();   // this block is in LDS; thread 0 has left the other buffer
        if (i0 > 0) hand_over(i0 - F, buf ^ 1);
        if (i0 + F < n_rows) issue(i0 + F, buf ^ 1);
        if (tid == 0) {
            const int cnt = min(F, n_rows - i0);
            const uint16_t *r = bt_rows + (size_t)buf * F * W;
            for (int f = 0; f < cnt; ++f, r += W) {
                s = r[s < P.Kcap ? at_states + s : at_clones + (s - P.Kcap)];
                walked[buf * kBtFrames + f] = (uint16_t)s;
            }
        }
    }
    __syncthreads();
    if (n_rows > 0) hand_over((n_rows - 1) / F * F, (n_rows - 1) / F & 1);
}

// Best path, rows kept whole (fb_best_linear_kernel): the two halves joined and followed.  The score and where it is attained as
// in fb_backtrace_kernel; from there a path's state at the next frame is the source of the largest of its state's terms, formed
// anew from that frame's row: the same additions as in the recursion, so the same largest (of equal ones the smallest source).
// One workgroup per sequence and half.  A step is a chain: where the state's arcs begin (LDS), the arcs (L2), their sources' scores
// (LDS: kTraceWalk waves walk), the largest over the workgroup; three waves bring the rows from memory straight into LDS, three frames ahead,
// one keeps the path and stores 64 frames of it at a time: a walking wave has no memory operation on its way but the arcs it waits for.
// Bound: the rows, read once (932 MB for 128 sequences of 100 to 500 frames over 6000 states: 366 us, 2.5 TB/s, while the
// longest sequences are left; four walking waves instead of eight, or one arc a trip instead of four, take the same time).
constexpr int kTraceWalk = 8, kTraceLoad = 3, kTraceRows = 4, kTraceThreads = (kTraceWalk + kTraceLoad + 1) * kWave;

__global__ __launch_bounds__(kTraceThreads) void fb_best_trace_kernel(const BestTraceParams P)
{
    extern __shared__ float tr_rows[];   // [kTraceRows][ld], then ptr, candidates
    const int b = blockIdx.x % P.B, half = blockIdx.x / P.B, tid = threadIdx.x;   // half 0: frames m .. 0, 1: m + 1 .. T - 1
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = min(max(P.lengths[b], 0), P.N), m = path_middle(T), K = P.K;
    const int64_t ld = P.ld;
    int32_t *prow = P.path + (size_t)b * P.N;
    if (half == 0)
        for (int n = T + tid; n < P.N; n += kTraceThreads) prow[n] = -1;
    if (T == 0) {
        if (half == 0 && tid == 0) P.score[b] = -INFINITY;
        return;
    }
    int32_t *const ptr = (int32_t *)(tr_rows + kTraceRows * ld);
    double *const red_v = (double *)(ptr + ((K + 2) & ~1));        // [waves]
    int32_t *const red_a = (int32_t *)(red_v + kTraceThreads / kWave);
    float *const cand_v = (float *)(red_a + kTraceThreads / kWave);   // [2][kTraceWalk]
    int32_t *const cand_s = (int32_t *)(cand_v + 2 * kTraceWalk);
    const int n_rows = half ? T - 1 - m : m;
    auto frame_of = [&](int i) { return half ? m + 1 + i : m - 1 - i; };   // the i-th row: frame of the state it decides
    // row i -> its place, by the loading waves
    const int n16 = (int)(ld / 4), loader = wave - kTraceWalk;
    const int mine = loader >= 0 && loader < kTraceLoad ? ((n16 + kWave - 1) / kWave - loader + kTraceLoad - 1) / kTraceLoad : 0;   // pieces of a row
    auto issue = [&](int i) {
        const float4 *row = (const float4 *)(P.rows + ((size_t)b * P.N + frame_of(i)) * ld);
        float4 *dst = (float4 *)(tr_rows + (i % kTraceRows) * ld);
        for (int p = loader; p * kWave < n16; p += kTraceLoad)
            if (p * kWave + lane < n16)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + p * kWave + lane),
                                                 (__attribute__((address_space(3))) void *)(dst + p * kWave), 16, 0, 0);
    };
    // all rows but the last `later` asked for have arrived
    auto arrived = [&](int later) {
        switch (later * mine) {   // (a wait for fewer than may be on their way is right as well)
        case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
        case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
        case 8: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
        case 10: asm volatile("s_waitcnt vmcnt(10)" ::: "memory"); break;
        case 12: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
        case 14: asm volatile("s_waitcnt vmcnt(14)" ::: "memory"); break;
        case 16: asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); break;
        case 18: asm volatile("s_waitcnt vmcnt(18)" ::: "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        }
    };

    // ---- the score and the path's state at frame m (both workgroups of a sequence find the same)
    double best = -INFINITY;
    int at = 0x7fffffff;
    auto take = [&](double v, int a) {
        if (v > best || (v == best && a < at)) { best = v; at = a; }
    };
    for (int k = tid; k < K; k += kTraceThreads) take((double)P.mid[0][(size_t)b * P.mid_ld + k] + (double)P.mid[1][(size_t)b * P.mid_ld + k], k);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const double v = __shfl_xor(best, o, 64);
        const int a = __shfl_xor(at, o, 64);
        take(v, a);
    }
    if (lane == 0) { red_v[wave] = best; red_a[wave] = at; }
    const int32_t *const gptr = P.ptr[half];
    for (int k = tid; k <= K; k += kTraceThreads) ptr[k] = gptr[k];
    __syncthreads();
    best = red_v[0]; at = red_a[0];
    for (int w = 1; w < kTraceThreads / kWave; ++w) take(red_v[w], red_a[w]);
    const bool none = !(best > -INFINITY);
    if (half == 0 && tid == 0) P.score[b] = none ? -INFINITY : (P.mid_off[0][b] + P.mid_off[1][b] + best) * kLn2;
    if (none) {
        for (int i = tid; i < (half ? n_rows : m + 1); i += kTraceThreads) prow[half ? m + 1 + i : i] = -1;
        return;
    }
    if (half == 0 && tid == 0) prow[m] = at;

    // ---- along the path
    int s = __builtin_amdgcn_readfirstlane(at);
    // what the waves have found in step i
    auto chosen = [&](int i) {
        const int c = (i & 1) * kTraceWalk;
        float v = cand_v[c];
        int a = cand_s[c];
#pragma unroll
        for (int w = 1; w < kTraceWalk; ++w) {
            const float vw = cand_v[c + w];
            const int aw = cand_s[c + w];
            const bool better = vw > v || (vw == v && aw < a);
            v = better ? vw : v;
            a = better ? aw : a;
        }
        return __builtin_amdgcn_readfirstlane(a);
    };
    if (wave < kTraceWalk) {
        const Arc *const arcs = P.arcs[half];
        __syncthreads();                                    // row 0
        for (int i = 0; i < n_rows; ++i) {
            const float *row = tr_rows + (i % kTraceRows) * ld;
            const int e0 = ptr[s], e1 = ptr[s + 1];
            float v = -INFINITY;
            int a = 0x7fffffff;
            auto look = [&](const Arc &arc) {
                const float x = row[arc.src] + arc.w;
                const bool better = x > v || (x == v && arc.src < a);
                v = better ? x : v;
                a = better ? arc.src : a;
            };
            // (behind the row's end a lane looks at its last arc again: what is asked for at once then takes one trip to the L2)
            constexpr int kStride = kTraceWalk * kWave, kAhead = 4;
            const bool any = e0 + wave * kWave < e1;        // (uniform) this wave has an arc
            if (any && e1 - e0 <= kStride) {
                look(arcs[min(e0 + tid, e1 - 1)]);
            } else if (any) {
                for (int e = e0 + tid; e - lane < e1; e += kAhead * kStride) {
                    Arc arc[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) arc[u] = arcs[min(e + u * kStride, e1 - 1)];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) look(arc[u]);
                }
            }
            float top = -INFINITY;
            int src = 0x7fffffff;
            if (any) {
                top = lane_value(wave_max_last(v), kWave - 1);
                src = group_all(v == top ? a : 0x7fffffff, 6, lane, [](int x, int y) { return min(x, y); });
            }
            if (lane == 0) {
                cand_v[(i & 1) * kTraceWalk + wave] = top;
                cand_s[(i & 1) * kTraceWalk + wave] = src;
            }
            lds_barrier();
            s = min(chosen(i), K - 1);                      // (the state's score is above zero-bar: a term of its row is)
        }
    } else if (loader < kTraceLoad) {
        for (int i = 0; i < min(kTraceRows - 1, n_rows); ++i) issue(i);
        arrived(n_rows >= kTraceRows - 1 ? kTraceRows - 2 : 0);
        __syncthreads();
        for (int i = 0; i < n_rows; ++i) {
            const bool more = i + kTraceRows - 1 < n_rows;
            if (more) issue(i + kTraceRows - 1);            // in the place of row i - 1
            arrived(more ? kTraceRows - 2 : 0);             // row i + 1 is there
            lds_barrier();
        }
    } else {
        int kept = 0;
        __syncthreads();
        for (int i = 0; i < n_rows; ++i) {
            lds_barrier();
            const int a = min(chosen(i), K - 1);
            kept = lane == (i & (kWave - 1)) ? a : kept;
            if ((i & (kWave - 1)) == kWave - 1 || i == n_rows - 1) {
                const int j = (i & ~(kWave - 1)) + lane;
                if (j <= i) prow[frame_of(j)] = kept;
            }
        }
    }
}


// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static int check_launch(const char *what)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FB_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    return FB_OK;
}

template <class Kern>
static int launch_rec(Kern kern, int nw, const RecParams &p, size_t lds_bytes, void *stream)
{
    if (lds_bytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return fail(FB_EHIP, std::string("hipFuncSetAttribute(LDS size): ") + hipGetErrorString(e));
    }
    const int32_t n_seq = p.order ? p.n_launch : p.B;
    hipLaunchKernelGGL(kern, dim3((unsigned)(n_seq * p.n_dir)), dim3(nw * kWave), lds_bytes, (hipStream_t)stream, p);
    return check_launch("recursion kernel launch");
}

typedef void (*rec_kernel_t)(const RecParams);

static rec_kernel_t linear_kernel_of(bool logs, int few, bool apart)
{
    if (apart)
        return few == kPFew ? (logs ? fb_linear_kernel<true, kPFew, true> : fb_linear_kernel<false, kPFew, true>)
               : few        ? (logs ? fb_linear_kernel<true, kPFewMost, true> : fb_linear_kernel<false, kPFewMost, true>)
                            : (logs ? fb_linear_kernel<true, 0, true> : fb_linear_kernel<false, 0, true>);
    return few == kPFew ? (logs ? fb_linear_kernel<true, kPFew, false> : fb_linear_kernel<false, kPFew, false>)
           : few        ? (logs ? fb_linear_kernel<true, kPFewMost, false> : fb_linear_kernel<false, kPFewMost, false>)
                        : (logs ? fb_linear_kernel<true, 0, false> : fb_linear_kernel<false, 0, false>);
}
static const void *linear_kernel(bool logs, int few, bool apart) { return (const void *)linear_kernel_of(logs, few, apart); }

bool recursion_fixed_available()
{
    // the fixed-buffer instantiation addresses LDS from 0: usable only while the kernel has no static LDS in front
    // of its dynamic array (a property of the build, looked up once)
    static const bool ok = [] {
        const void *kernels[] = {(const void *)fb_recursion_kernel<kNWShared, float, false, kXsFixed>,
                                 (const void *)fb_recursion_kernel<kNWShared, float, false, kXsFixed, true>,
                                 linear_kernel(false, 0, false), linear_kernel(false, kPFew, false), linear_kernel(false, kPFewMost, false),
                                 linear_kernel(true, 0, false), linear_kernel(true, kPFew, false), linear_kernel(true, kPFewMost, false),
                                 linear_kernel(false, 0, true), linear_kernel(false, kPFew, true), linear_kernel(false, kPFewMost, true),
                                 linear_kernel(true, 0, true), linear_kernel(true, kPFew, true), linear_kernel(true, kPFewMost, true),
                                 (const void *)fb_leaky_linear_kernel<0>, (const void *)fb_leaky_linear_kernel<kPFew>,
                                 (const void *)fb_leaky_linear_kernel<kPFewMost>, (const void *)fb_best_linear_kernel<0>,
                                 (const void *)fb_best_linear_kernel<kPFew>, (const void *)fb_best_linear_kernel<kPFewMost>};
        for (const void *k : kernels) {
            hipFuncAttributes attr{};
            if (hipFuncGetAttributes(&attr, k) != hipSuccess || attr.sharedSizeBytes != 0) return false;
        }
        return true;
    }();
    return ok;
}

// kPFew or kPFewMost if every direction's plan keeps its units in that many places in registers, else 0
static int few_units(const RecParams &p)
{
    int most = 0;
    for (int i = 0; i < p.n_dir; ++i) most = p.dir[i].prob.paired ? std::max(most, p.dir[i].prob.max_units) : kPMaxUnits;
    return most <= kPFew ? kPFew : most <= kPFewMost ? kPFewMost : 0;
}

int launch_recursion(int nw, bool f64, bool tropical, const RecParams &p, size_t lds_bytes, void *stream)
{
    if (p.xs_fixed) {   // fixed-length state buffers: large graphs with float vectors only
        if (p.xs_fixed != kXsFixed || nw != kNWShared || f64 || tropical) return fail(FB_EHIP, "internal error: fixed-buffer launch");
        if (p.linear_p) {
            if (!p.shared || p.linear_w) return fail(FB_EHIP, "internal error: probability-domain launch");
            bool logs = false;
            for (int i = 0; i < p.n_dir; ++i) logs = logs || (p.dir[i].out && !p.dir[i].out_linear);
            for (int i = 0; i < p.n_dir; ++i) {
                if (!p.dir[i].prob.units) return fail(FB_EHIP, "internal error: probability-domain launch without its plan");
                lds_bytes = std::max(lds_bytes, probability_lds_bytes(p.D, p.dir[i].backward != 0 || logs));
            }
            if (lds_bytes > kLdsBytes) return fail(FB_EHIP, "internal error: probability-domain launch beyond the on-chip memory");
            bool apart = false;
            for (int i = 0; i < p.n_dir; ++i) apart = apart || p.dir[i].prob.apart;
            const rec_kernel_t kern = linear_kernel_of(logs, few_units(p), apart);
            return launch_rec(kern, nw, p, lds_bytes, stream);
        }
        if (p.linear_w) return launch_rec(fb_recursion_kernel<kNWShared, float, false, kXsFixed, true>, nw, p, lds_bytes, stream);
        return launch_rec(fb_recursion_kernel<kNWShared, float, false, kXsFixed>, nw, p, lds_bytes, stream);
    }
    if (p.linear_w) return fail(FB_EHIP, "internal error: linear weights without fixed buffers");
    if (tropical) {
        if (nw == kNWShared)
            return f64 ? launch_rec(fb_recursion_kernel<kNWShared, double, true, 0>, nw, p, lds_bytes, stream)
                       : launch_rec(fb_recursion_kernel<kNWShared, float, true, 0>, nw, p, lds_bytes, stream);
        return f64 ? launch_rec(fb_recursion_kernel<kNWSmall, double, true, 0>, nw, p, lds_bytes, stream)
                   : launch_rec(fb_recursion_kernel<kNWSmall, float, true, 0>, nw, p, lds_bytes, stream);
    }
    if (nw == kNWShared)
        return f64 ? launch_rec(fb_recursion_kernel<kNWShared, double, false, 0>, nw, p, lds_bytes, stream)
                   : launch_rec(fb_recursion_kernel<kNWShared, float, false, 0>, nw, p, lds_bytes, stream);
    return f64 ? launch_rec(fb_recursion_kernel<kNWSmall, double, false, 0>, nw, p, lds_bytes, stream)
               : launch_rec(fb_recursion_kernel<kNWSmall, float, false, 0>, nw, p, lds_bytes, stream);
}

int launch_best_linear(const RecParams &p, void *stream)
{
    for (int i = 0; i < p.n_dir; ++i)
        if (!p.shared || !p.dir[i].prob.units || !p.dir[i].mid || !p.dir[i].out) return fail(FB_EHIP, "internal error: best-path launch without its plan");
    const size_t lds = probability_lds_bytes(p.D, false);
    if (lds > kLdsBytes || !recursion_fixed_available()) return fail(FB_EHIP, "internal error: best-path launch beyond the on-chip memory");
    const int few = few_units(p);
    auto kern = few == kPFew ? fb_best_linear_kernel<kPFew> : few ? fb_best_linear_kernel<kPFewMost> : fb_best_linear_kernel<0>;
    return launch_rec(kern, kNWShared, p, lds, stream);
}

size_t leaky_linear_lds_bytes(int32_t K, int32_t Ccap, int32_t D, bool backward)
{
    const size_t XL = ((size_t)K + (size_t)Ccap + 1 + 3) & ~(size_t)3;
    return (size_t)kXbStride + (XL * (backward ? 4 : 2) + kProbWords + 3 * (size_t)prob_row_floats(D)) * 4;
}

int launch_leaky_linear(const RecParams &p, int32_t *gave_up, void *stream)
{
    size_t lds = 0;
    for (int i = 0; i < p.n_dir; ++i) {
        if (!p.dir[i].prob.units || !p.dir[i].rank1 || !p.dir[i].fmt) return fail(FB_EHIP, "internal error: leaky-HMM launch without its plan");
        lds = std::max(lds, leaky_linear_lds_bytes(p.Kcap, p.dir[i].prob.Ccap, p.D, p.dir[i].backward != 0));
    }
    if (lds > kLdsBytes || !recursion_fixed_available()) return fail(FB_EHIP, "internal error: leaky-HMM launch beyond the on-chip memory");
    const int few = few_units(p);
    auto kern = few == kPFew ? fb_leaky_linear_kernel<kPFew> : few ? fb_leaky_linear_kernel<kPFewMost> : fb_leaky_linear_kernel<0>;
    const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return fail(FB_EHIP, std::string("hipFuncSetAttribute(LDS size): ") + hipGetErrorString(e));
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.B * p.n_dir)), dim3(kNWShared * kWave), lds, (hipStream_t)stream, p, gave_up);
    return check_launch("leaky-HMM recursion launch");
}

size_t probability_lds_bytes(int32_t D, bool staged)
{
    return (size_t)kXbStride + ((size_t)kXsFixed * (staged ? 3 : 1) + kProbWords + 3 * (size_t)prob_row_floats(D)) * 4;
}

unsigned int linear_restarts()
{
    unsigned int n = 0;
    if (hipMemcpyFromSymbol(&n, HIP_SYMBOL(g_linear_restarts), sizeof(n)) != hipSuccess) return 0;
    return n;
}

int launch_backtrace(const BacktraceParams &p, void *stream)
{
    // rows of the sequence with the most columns: its states and the clone slots
    BacktraceParams q = p;
    if ((p.bp_ld & 7) != 0 || ((uintptr_t)p.bp & 15) != 0) return fail(FB_EHIP, "internal error: back-pointer rows are not in 16-byte pieces");
    const size_t row_bytes = ((size_t)p.Kcap + (size_t)p.Ccap + 32) * sizeof(uint16_t);   // both spans rounded out to whole pieces
    const size_t extra = kBtThreads / kWave * (sizeof(double) + sizeof(uint32_t)) + 2 * kBtFrames * sizeof(uint16_t);
    auto fit = [&](size_t room, int most) { return (int32_t)std::max<size_t>(1, std::min<size_t>((size_t)most, (room - extra) / (2 * row_bytes))); };   // two buffers
    // Short rows: as many as 64 KB hold, since a block costs a trip to memory whatever it holds; long ones: a block of
    // 8 frames keeps a compute unit's share of the memory rate busy, more only take LDS.
    q.frames = std::max(fit(kBtSmallBytes, kBtFrames), fit(kLdsBytes - kLdsReserve, kBtLargeFrames));
    const size_t lds_bytes = 2 * (size_t)q.frames * row_bytes + extra;
    if (lds_bytes > kLdsBytes) return fail(FB_EUNSUPPORTED, "backtrace: a row of back-pointers exceeds the on-chip memory");
    if (lds_bytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)fb_backtrace_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return fail(FB_EHIP, std::string("hipFuncSetAttribute(LDS size): ") + hipGetErrorString(e));
    }
    hipLaunchKernelGGL(fb_backtrace_kernel, dim3((unsigned)(2 * p.B)), dim3(kBtThreads), lds_bytes, (hipStream_t)stream, q);
    return check_launch("backtrace kernel launch");
}

size_t best_trace_lds_bytes(int32_t K)
{
    const size_t ld = ((size_t)K + 3) & ~(size_t)3;
    return kTraceRows * ld * 4 + (((size_t)K + 2) & ~(size_t)1) * 4 + kTraceThreads / kWave * 12 + 2 * kTraceWalk * 8;
}

int launch_best_trace(const BestTraceParams &p, void *stream)
{
    const size_t lds = best_trace_lds_bytes(p.K);
    if (lds > kLdsBytes || (p.ld & 3) != 0 || ((uintptr_t)p.rows & 15) != 0) return fail(FB_EHIP, "internal error: best-path trace launch");
    const hipError_t e = hipFuncSetAttribute((const void *)fb_best_trace_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return fail(FB_EHIP, std::string("hipFuncSetAttribute(LDS size): ") + hipGetErrorString(e));
    hipLaunchKernelGGL(fb_best_trace_kernel, dim3((unsigned)(2 * p.B)), dim3(kTraceThreads), lds, (hipStream_t)stream, p);
    return check_launch("best-path trace kernel launch");
}

int launch_posteriors(const PostParams &p, size_t lds_bytes, void *stream)
{
    const dim3 grid((unsigned)((p.N + p.frames_per_block - 1) / p.frames_per_block), (unsigned)(p.order ? p.n_launch : p.B));
    if (lds_bytes > 64 * 1024) {
        const hipError_t e =
            hipFuncSetAttribute((const void *)fb_posterior_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return fail(FB_EHIP, std::string("hipFuncSetAttribute(LDS size): ") + hipGetErrorString(e));
    }
    hipLaunchKernelGGL(fb_posterior_kernel, grid, dim3(kPostThreads), lds_bytes, (hipStream_t)stream, p);
    return check_launch("posterior kernel launch");
}

bool gradient_kernel_applies(const PostParams &p)
{
    if (!p.pdf_out || p.accumulate) return false;
    const bool offsets = p.cum_a && p.cum_b && p.logz;
    if (p.n_graph == 1) {   // the shared graph's share alone: no numerators
        const PostGraph &d = p.g[0];
        // without the offsets of the rows only rows of logarithms (no format flags), relative to each frame's maximum
        if (!offsets && (p.cum_a || p.cum_b || p.logz || d.fmt_a || d.fmt_b)) return false;
        // (rows that are not in whole 16-byte pieces are read piece by piece and need no padding)
        const bool pieces16 = (d.ld & 3) == 0 && d.ld >= ((d.Kcap + 3) & ~3) && (((uintptr_t)d.a | (uintptr_t)d.b) & 15) == 0;
        const bool any_rows = d.ld >= d.Kcap && (((uintptr_t)d.a | (uintptr_t)d.b) & 3) == 0;
        return d.shared && !d.f64 && !d.state_post && d.pdfs.pos && (pieces16 || any_rows) &&
               d.Kcap <= kGradMain * 4 * kGradU && p.D <= kGradMain * kGradPdf;
    }
    if (p.n_graph != 2 || !offsets) return false;
    const PostGraph &d = p.g[0], &n = p.g[1];
    return d.shared && !d.f64 && !d.state_post && d.pdfs.pos && (d.ld & 3) == 0 && d.ld >= ((d.Kcap + 3) & ~3) &&
           d.Kcap <= kGradMain * 4 * kGradU &&
           (((uintptr_t)d.a | (uintptr_t)d.b) & 15) == 0 && p.D <= kGradMain * kGradPdf && !n.shared && !n.state_post &&
           n.Kcap <= kGradNumK && n.Rcap <= kGradNumK;
}

size_t gradient_lds_bytes(const PostParams &p)
{
    const PostGraph &d = p.g[0], &n = p.g[1];
    const size_t nR = p.n_graph == 2 ? (size_t)n.Rcap : 0, nK = p.n_graph == 2 ? (size_t)n.Kcap : 0;   // one graph: no numerator tables
    return 256 + (2 * ((size_t)((d.Kcap + 3) & ~3) + kGradSlack) + 2 * nR + nK) * 4 + ((size_t)((p.D + 1) & ~1) + nR * 2 + 1 + nK + 3) / 2 * 4;
}

int launch_gradient(const PostParams &p, size_t lds_bytes, void *stream)
{
    const dim3 grid((unsigned)((p.N + p.frames_per_block - 1) / p.frames_per_block), (unsigned)(p.order ? p.n_launch : p.B));
    auto kern = p.n_graph == 2 && p.g[1].f64 ? fb_grad_kernel<double> : fb_grad_kernel<float>;
    if (lds_bytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return fail(FB_EHIP, std::string("hipFuncSetAttribute(LDS size): ") + hipGetErrorString(e));
    }
    hipLaunchKernelGGL(kern, grid, dim3(kGradThreads), lds_bytes, (hipStream_t)stream, p);
    return check_launch("gradient kernel launch");
}

bool num_add_kernel_applies(const PostParams &p)
{
    if (p.n_graph != 1 || !p.accumulate || !p.pdf_out) return false;
    const PostGraph &n = p.g[0];
    return !n.shared && !n.state_post && n.Kcap <= kGradNumK && n.Rcap <= kGradNumK;
}

int launch_num_add(const PostParams &p, void *stream)
{
    const PostGraph &n = p.g[0];
    const size_t lds_bytes = (size_t)n.Kcap * 4 + ((size_t)n.Rcap * 2 + 1 + (size_t)n.Kcap + 3) / 2 * 4;
    const dim3 grid((unsigned)((p.N + p.frames_per_block - 1) / p.frames_per_block), (unsigned)(p.order ? p.n_launch : p.B));
    auto kern = n.f64 ? fb_num_add_kernel<double> : fb_num_add_kernel<float>;
    hipLaunchKernelGGL(kern, grid, dim3(kWave), lds_bytes, (hipStream_t)stream, p);
    return check_launch("numerator kernel launch");
}

// Does nothing: a launch whose only effect is that what follows it on its stream starts one launch latency later.
__global__ __launch_bounds__(64) void fb_delay_kernel() {}

// *flag = whether the counter has reached `need` (a progress counter of a launch that may still be running)
__global__ __launch_bounds__(64) void fb_decide_kernel(const uint32_t *count, uint32_t need, int32_t *flag)
{
    if (threadIdx.x == 0) *flag = *(const volatile uint32_t *)count >= need ? 1 : 0;
}

__global__ __launch_bounds__(64) void fb_mark_kernel(uint32_t *word)
{
    if (threadIdx.x == 0) *word = 1u;
}

int launch_mark(uint32_t *word, void *stream)
{
    hipLaunchKernelGGL(fb_mark_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, word);
    return check_launch("mark kernel launch");
}

int launch_decide(const uint32_t *count, uint32_t need, int32_t *flag, void *stream)
{
    hipLaunchKernelGGL(fb_decide_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, count, need, flag);
    return check_launch("decide kernel launch");
}

int launch_delay(void *stream)
{
    hipLaunchKernelGGL(fb_delay_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream);
    return check_launch("delay kernel launch");
}

int launch_order(const int32_t *lengths, int32_t B, int32_t N, int32_t *order, uint32_t *done, void *stream)
{
    hipLaunchKernelGGL(fb_order_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, (hipStream_t)stream, lengths, B, N, order, done);
    return check_launch("order kernel launch");
}

int launch_loss(const double *zn, const double *zd, const int32_t *lengths, int32_t B, double *loss, void *stream)
{
    hipLaunchKernelGGL(fb_loss_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, zn, zd, lengths, B, loss);
    return check_launch("loss kernel launch");
}

}  // namespace fb
