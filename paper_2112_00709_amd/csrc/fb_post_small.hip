// State and pdf posteriors (Eq. 15) of small (sub-)graphs: at most 1024 states each, of one graph (shared or packed) or
// of a shared graph and packed ones, each with its sign (Eq. 17).  What fb_posterior_kernel computes, for the sizes where
// that kernel's time is its chain: a workgroup of 512 threads takes its frames one after the other with six barriers
// each, most threads without a state.
//
// Here a wave takes a frame by itself: a lane holds up to U states of the row, maximum and sum are reductions over the
// wave, the exponentials go to the wave's own LDS in pdf order (a pdf's states are neighbours, the place of a lane's
// states is kept in registers for all its frames), and no barrier follows the one behind the tables.  Four waves share
// the tables; a wave takes F frames, as many as leave about two workgroups per compute unit.  Sums are formed in a fixed
// order.  A shared graph has a row for every pdf and needs no list of the rows it has: 300 states, 3000 pdfs, 128 x 300 frames
// 369 -> 185 us without the room for one (half the chip's waves had no place).  Measured (three-call forward-backward, this call alone): 16 states, 1 x 50 frames, 19 -> 5.8 us; 32
// chains of 30-120 states, 3.0 k frames, with state posteriors 39 -> 7.6 us; 701 states, 97 pdfs, 3.1 k frames,
// with state posteriors 46 -> 20 us.  Bound: launch and HBM latency in the first, the row traffic in the last.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "fb_device.h"
#include "fb_internal.h"

namespace fb {

namespace {

constexpr int kPostWaves = 4;

struct PostSmallLds {      // bytes of the parts of a workgroup's LDS; the kernel and its launch agree through this
    size_t ptr[2], nidx, tb[2], nval, total;
    __host__ __device__ explicit PostSmallLds(const PostParams &P)
    {
        size_t at = 0;
        const bool two = P.n_graph == 2, packed = two || !P.g[0].shared;   // packed: the last graph's rows are a selection of the pdfs
        ptr[0] = 0; at = ((size_t)P.g[0].Rcap + 2) / 2 * 4;
        ptr[1] = at; at += two ? ((size_t)P.g[1].Rcap + 2) / 2 * 4 : 0;
        nidx = at; at += packed ? ((size_t)P.D + 1) / 2 * 4 : 0;
        tb[0] = at; at += (size_t)kPostWaves * (size_t)P.g[0].Kcap * 4;
        tb[1] = at; at += two ? (size_t)kPostWaves * (size_t)P.g[1].Kcap * 4 : 0;
        nval = at; at += packed ? (size_t)kPostWaves * (size_t)(two ? P.g[1].Rcap : P.g[0].Rcap) * 4 : 0;
        total = at;
    }
};

}  // namespace

template <int U>
__global__ __launch_bounds__(kPostWaves * kWave) void fb_post_small_kernel(const PostParams P)
{
    extern __shared__ double lds_raw[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = P.order ? P.order[P.rank0 + blockIdx.y] : blockIdx.y;
    const int T = min(max(P.lengths[b], 0), P.N);
    const int F = P.frames_per_block / kPostWaves, n0 = blockIdx.x * P.frames_per_block;
    const PostSmallLds at(P);
    char *const lds = (char *)lds_raw;
    uint16_t *const nidx = (uint16_t *)(lds + at.nidx);
    const bool two = P.n_graph == 2;
    float *const nval = (float *)(lds + at.nval) + (size_t)wave * (two ? P.g[1].Rcap : P.g[0].Rcap);
    const bool packed_last = two || !P.g[0].shared;
    PdfSub ps[2] = {};
    uint16_t pos[2][U];                                     // places of the lane's states in pdf order
    // (loops over the two graphs are unrolled: what is indexed by the graph stays in registers)
#pragma unroll
    for (int gi = 0; gi < 2; ++gi)
        if (gi < P.n_graph) ps[gi] = P.g[gi].pdfs.sub[P.g[gi].shared ? 0 : b];
    if (n0 < T) {                                           // the tables: only if a real frame follows
        if (packed_last)
            for (int d = tid; d < P.D; d += kPostWaves * kWave) nidx[d] = 0;
#pragma unroll
        for (int gi = 0; gi < 2; ++gi) {
            if (gi >= P.n_graph) break;
            const PostGraph &G = P.g[gi];
            uint16_t *ptr = (uint16_t *)(lds + at.ptr[gi]);
            // (the exponentials' buffers of the four waves hold the inverse of the table for the moment)
            uint16_t *inv = (uint16_t *)(lds + at.tb[gi]);
            for (int r = tid; r <= ps[gi].n_rows; r += kPostWaves * kWave) ptr[r] = G.pdfs.row_ptr[ps[gi].ptr0 + r];
            for (int i = tid; i < ps[gi].K; i += kPostWaves * kWave) inv[G.pdfs.states[ps[gi].st0 + i]] = (uint16_t)i;
        }
        __syncthreads();
        if (packed_last) {
            const uint16_t *row_pdf = two ? P.g[1].pdfs.row_pdf : P.g[0].pdfs.row_pdf;
            const int row0 = two ? ps[1].row0 : ps[0].row0, n_rows = two ? ps[1].n_rows : ps[0].n_rows;
            for (int r = tid; r < n_rows; r += kPostWaves * kWave) nidx[row_pdf[row0 + r]] = (uint16_t)(r + 1);
        }
#pragma unroll
        for (int gi = 0; gi < 2; ++gi)
            if (gi < P.n_graph) {
                const uint16_t *inv = (const uint16_t *)(lds + at.tb[gi]);
#pragma unroll
                for (int u = 0; u < U; ++u) pos[gi][u] = u * kWave + lane < ps[gi].K ? inv[u * kWave + lane] : (uint16_t)0;
            }
        __syncthreads();
    }
    for (int f = 0; f < F; ++f) {
        const int n = n0 + f * kPostWaves + wave;
        if (n >= P.N) break;
        float *prow = P.pdf_out ? P.pdf_out + ((size_t)b * P.N + n) * P.D : nullptr;
        if (n >= T) {                                       // padded frame: zeros
            if (prow)
                for (int d = lane; d < P.D; d += kWave) prow[d] = 0.0f;
#pragma unroll
            for (int gi = 0; gi < 2; ++gi) {
                if (gi >= P.n_graph) break;
                const PostGraph &G = P.g[gi];
                if (!G.state_post) continue;
                float *srow = G.shared ? G.state_post + ((size_t)b * P.N + n) * ps[gi].K : G.state_post + (size_t)n * G.Ktot + ps[gi].k0;
                for (int k = lane; k < ps[gi].K; k += kWave) srow[k] = 0.0f;
            }
            continue;
        }
        float scale[2];
        // exponentials of the frame's log posteriors (a + b), relative to the largest, in pdf order -> tb; the state
        // posteriors; sign / sum -> scale
        auto states = [&](auto gi_c, auto type) __attribute__((always_inline)) {
            constexpr int gi = decltype(gi_c)::value;
            typedef decltype(type) IT;
            const PostGraph &G = P.g[gi];
            const int K = ps[gi].K;
            const size_t row = G.shared ? ((size_t)b * P.N + n) * G.ld : (size_t)n * G.Ktot + ps[gi].k0;
            const IT *a = (const IT *)G.a + row, *bb = (const IT *)G.b + row;
            float *tb = (float *)(lds + at.tb[gi]) + (size_t)wave * G.Kcap;
            IT t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = min(u * kWave + lane, K - 1);   // (a lane without a state takes the last one again, and counts nothing)
                t[u] = u * kWave < K ? (a[k] + bb[k]) * (IT)G.in_scale : (IT)(-INFINITY);
            }
            IT mx = t[0];
#pragma unroll
            for (int u = 1; u < U; ++u) mx = tmax(mx, t[u]);
            mx = wave_max(mx);
            const bool mass = mx != (IT)(-INFINITY);
            float e[U], sum = 0.0f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                e[u] = mass && u * kWave + lane < K ? fexp2((float)(t[u] - mx)) : 0.0f;
                sum += e[u];
            }
            sum = wave_sum(sum);
            const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;
            scale[gi] = G.sign * inv;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the frame before has been read
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u * kWave + lane < K) tb[pos[gi][u]] = e[u];
            if (G.state_post) {
                float *srow = G.shared ? G.state_post + ((size_t)b * P.N + n) * K : G.state_post + (size_t)n * G.Ktot + ps[gi].k0;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (u * kWave + lane < K) srow[u * kWave + lane] = e[u] * inv;
            }
        };
        // put(row, sum over the states of the graph's pdf row) for every row; lanes share a row when there are few of them
        auto rows = [&](auto gi_c, auto put) __attribute__((always_inline)) {
            constexpr int gi = decltype(gi_c)::value;
            const uint16_t *ptr = (const uint16_t *)(lds + at.ptr[gi]);
            const float *tb = (const float *)(lds + at.tb[gi]) + (size_t)wave * P.g[gi].Kcap;
            const int n_rows = ps[gi].n_rows;
            int tpr = 1;
            while (tpr < 16 && n_rows * tpr * 2 <= kWave) tpr *= 2;
            const int part = lane & (tpr - 1), per = kWave / tpr;
            for (int r0 = 0; r0 < n_rows; r0 += per) {
                const int r = r0 + lane / tpr;
                const int lo = r < n_rows ? ptr[r] : 0, hi = r < n_rows ? ptr[r + 1] : 0;
                float acc = 0.0f;
                for (int i = lo + part; i < hi; i += 4 * tpr) {   // four at a time, all read before any is added
                    float v[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = tb[min(i + j * tpr, hi - 1)];
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc += i + j * tpr < hi ? v[j] : 0.0f;
                }
                for (int o = 1; o < tpr; o <<= 1) acc += __shfl_xor(acc, o, kWave);
                if (part == 0 && r < n_rows) put(r, acc);
            }
        };
        const std::integral_constant<int, 0> first;
        const std::integral_constant<int, 1> second;
        if (P.g[0].f64) states(first, 0.0);
        else states(first, 0.0f);
        if (P.n_graph == 2) {
            if (P.g[1].f64) states(second, 0.0);
            else states(second, 0.0f);
        }
        if (!prow) continue;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (packed_last) {
            if (P.n_graph == 2) rows(second, [&](int r, float acc) { nval[r] = acc * scale[1]; });
            else rows(first, [&](int r, float acc) { nval[r] = acc * scale[0]; });
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        if (P.g[0].shared) {
            rows(first, [&](int d, float acc) {             // (a shared graph has a row for every pdf)
                float v = acc * scale[0];
                if (packed_last && nidx[d]) v += nval[nidx[d] - 1];
                prow[d] = v;
            });
        } else {
            for (int d = lane; d < P.D; d += kWave) prow[d] = nidx[d] ? nval[nidx[d] - 1] : 0.0f;
        }
    }
}

bool post_small_applies(const PostParams &p)
{
    if (p.accumulate || p.fused) return false;
    if (p.n_graph == 2 && (!p.g[0].shared || p.g[1].shared)) return false;
    for (int i = 0; i < p.n_graph; ++i)
        if (p.g[i].Kcap > kSmallStates || p.g[i].fmt_a || p.g[i].fmt_b) return false;
    // One shared graph of many states and pdfs, many frames: the workgroup-wide kernels read a row wider and keep fewer copies of
    // it.  128 x 300 frames, this kernel / the one that takes the call otherwise: 1000 states, 2000 pdfs 317 / 288 us; 600, 3000
    // 331 / 303; on this side of the line 600, 2000 264 / 288; 1000, 1000 239 / 275; 300, 3000 185 / 293.  16 x 200 frames, 1000
    // states, 3000 pdfs: 32 / 36.
    const int64_t frames = (int64_t)(p.order ? p.n_launch : p.B) * p.N;
    if (p.n_graph == 1 && p.g[0].shared && (int64_t)p.g[0].Kcap * p.D > 1500000 && frames > 8192) return false;
    return PostSmallLds(p).total <= 64 * 1024;              // (two workgroups and more on a compute unit)
}

int launch_post_small(const PostParams &p, void *stream)
{
    PostParams q = p;
    const int32_t n_seq = p.order ? p.n_launch : p.B;
    // frames per wave: as few as leave about two workgroups for each of 256 compute units
    const int64_t frames = (int64_t)n_seq * p.N;
    const int32_t F = (int32_t)std::min<int64_t>(8, std::max<int64_t>(1, frames / (kPostWaves * 512)));
    q.frames_per_block = F * kPostWaves;
    const dim3 grid((unsigned)((p.N + q.frames_per_block - 1) / q.frames_per_block), (unsigned)n_seq);
    int32_t K = 0;
    for (int i = 0; i < p.n_graph; ++i) K = std::max(K, p.g[i].Kcap);
    const size_t lds = PostSmallLds(p).total;
    auto kern = K <= kWave ? fb_post_small_kernel<1> : K <= 2 * kWave ? fb_post_small_kernel<2> : K <= 4 * kWave ? fb_post_small_kernel<4>
              : K <= 8 * kWave ? fb_post_small_kernel<8> : fb_post_small_kernel<16>;
    hipLaunchKernelGGL(kern, grid, dim3(kPostWaves * kWave), lds, (hipStream_t)stream, q);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? FB_OK : fail(FB_EHIP, std::string("small-graph posterior kernel launch: ") + hipGetErrorString(e));
}

}  // namespace fb
