// The alpha / beta recursions (Eq. 13-14) and their best-path form for small (sub-)graphs with vectors in double:
// numerator chains, alignment and label-sequence graphs, phone loops.
//
// A step of such a graph is a few hundred additions; what it costs is the length of the chain of dependent
// operations from one vector to the next.  The kernel keeps everything off that chain that need not be on it:
//   * No normalisation.  Exponentials act on differences of two terms, and a double holds a log value of 10^4 to
//     10^-12, so the vector is carried as it is.  The shift that makes float rows keep their resolution (a row's own
//     largest entry) is taken by the waves that write rows out.  That is for emissions as networks make them: a sequence
//     with an emission that is finite and larger than kLarge in size - a mask, of -1e20 or of the type's lowest value, say -
//     is done over (at once, if one is in the first frame) in a plain form that takes the previous vector's largest entry off
//     at every step, so that the frames before and behind such a frame keep their resolution.  So is every sequence of a
//     graph with weights of that size.  Calls with such emissions in every frame, against the general kernel and (in
//     brackets) against ordinary emissions: fb_alpha, fb_beta and fb_posteriors of 16 states over 50 frames 121 -> 118 us
//     (41), of 32 chains 283 -> 322 (70), of 701 states 878 -> 1063 (525; with the sums on probabilities
//     first, fb_small_linear.hip, 1120 and 285); best path of 32 label sequences 252 -> 139 (53).
//   * (A few scalars of the variants of 24 and 32 slices, and 13 vector registers of the best path's of 32, sit elsewhere.)
//     The arcs, targets and pdf ids of a lane sit in registers for the whole time loop (fb_small.cpp); a lane asks for
//     the emissions of its rows kAhead frames at a time, one such group ahead, straight into registers, so a step touches LDS for the gathers
//     and the new vector only.
//   * Rows leave through further waves of the workgroup, which read them out of a ring of LDS rows.  With one
//     computing wave the ring holds blocks of 8 frames and there is a barrier every 8 frames; with more of them the
//     barrier of every step that they need among themselves serves the writers too.
// The chain of a step is then: LDS read, add the weight, maximum / difference, one exponential, one logarithm, add
// the emission, LDS write (and the barrier).
//
// Zero-bar is carried as a number: start weights, arc weights and emissions of zero-bar (or below) are kZero = -1e36, so
// every sum is finite and no step meets inf - inf (a state that stays at zero-bar falls by that much a step, which a
// double takes); what lies below kZeroOut = -1e30 counts as zero-bar, as in the general kernel.  Nothing is clamped behind
// the emissions: a NaN among them (not a legal input, but what a diverged network hands over) is in log Z and the rows as
// it is in the general kernel's.  The best path has no differences of terms: zero-bar is -inf there, any finite score
// counts, and a state whose score is NaN is never taken.
//
// Measured per direction, against the general kernel with 4 waves (fb_recursion_kernel<4, double>): 32 chains of 30-120
// states over at most 144 frames 124 -> 29 us (of which the computing wave 24); a 16-state graph over 50 frames 55 -> 12
// (no row over several lanes) or 18 us; 701 states, 3.5 k arcs over at most 211 frames 442 -> 240 us; best path through 32
// label-sequence graphs of 21-161 states, 209 frames, 194 -> 64 us, and 40 us from both ends (fb_viterbi).  What bounds it: the latency of that chain (310
// clocks a step with one computing wave and two arcs a row); with 16 slices and more the issue of double arithmetic.
//
// Sums over shared graphs that mix run on probabilities instead (fb_small_linear.hip).
//
// Variants <NC, R, TM>: NC computing waves of R slices each, TM arcs per lane; the smallest that holds the batch's
// largest sub-graph is launched.
#include "fb_small_run.h"

namespace fb {

template <int NC, int R, int TM, bool TROP>
__global__ __launch_bounds__((NC + SmallShape<NC, R>::NIO) * kWave) void fb_small_kernel(const RecParams P)
{
    extern __shared__ double lds_raw[];
    if (P.started && threadIdx.x == 0) atomicAdd(P.started, 1u);   // this workgroup has its place on a compute unit
    int b, which;
    resolve_sequence<NC>(P, lds_raw, b, which);
    small_run<NC, R, TM, TROP, SmallShape<NC, R>::NIO>(P, (uint64_t)__builtin_amdgcn_kernarg_segment_ptr(), lds_raw, b, which);
    count_done(P);
}

template <int NC, int R, int TM, bool TROP>
static int launch_variant(const RecParams &p, void *stream)
{
    using S = SmallShape<NC, R>;
    bool backward = false;
    for (int i = 0; i < p.n_dir; ++i) backward = backward || p.dir[i].backward != 0;
    const size_t lds = S::lds_bytes(backward, TROP);
    static_assert(S::lds_bytes(true, TROP) <= 64 * 1024, "on-chip memory of a launch without a raised limit");
    const int32_t n_seq = p.order ? p.n_launch : p.B;
    hipLaunchKernelGGL((fb_small_kernel<NC, R, TM, TROP>), dim3((unsigned)(n_seq * p.n_dir)), dim3((NC + S::NIO) * kWave), lds, (hipStream_t)stream, p);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? FB_OK : fail(FB_EHIP, std::string("small-graph kernel launch: ") + hipGetErrorString(e));
}

template <int TM, bool TROP>
static int launch_size(const RecParams &p, int slices, void *stream)
{
    if (slices <= 1) return launch_variant<1, 1, TM, TROP>(p, stream);
    if (slices <= 2) return launch_variant<1, 2, TM, TROP>(p, stream);
    if (slices <= 4) return launch_variant<2, 2, TM, TROP>(p, stream);
    if (slices <= 8) return launch_variant<4, 2, TM, TROP>(p, stream);
    if (slices <= 16) return launch_variant<8, 2, TM, TROP>(p, stream);
    if (slices <= 24) return launch_variant<8, 3, TM, TROP>(p, stream);
    if (slices <= kSmallMaxSlices) return launch_variant<8, 4, TM, TROP>(p, stream);
    return fail(FB_EHIP, "internal error: small-graph launch");
}

int launch_small(const RecParams &p, int tm, int slices, bool tropical, void *stream)
{
    for (int i = 0; i < p.n_dir; ++i)
        if (!p.dir[i].small.arcs || (tropical && (p.dir[i].out || p.dir[i].off || p.dir[i].cum))) return fail(FB_EHIP, "internal error: small-graph launch without its plan, or best-path rows");
    if (p.Kcap > kSmallStates || (tm != 2 && tm != 4)) return fail(FB_EHIP, "internal error: small-graph launch");
    if (tm == 2) return tropical ? launch_size<2, true>(p, slices, stream) : launch_size<2, false>(p, slices, stream);
    return tropical ? launch_size<4, true>(p, slices, stream) : launch_size<4, false>(p, slices, stream);
}

}  // namespace fb
