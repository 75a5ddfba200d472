// Host-side construction of the plan the small-graph recursion kernel walks (fb_small.hip), its bounds check and its
// interpretation on the host for tests.
//
// The product is the one of fb_sell.cpp (row j gathers the arcs that enter, or leave, state j), for (sub-)graphs of at
// most 1024 states and a few thousand arcs with vectors in double.  Shape of the plan:
//   * A slice is 64 lanes of which each holds `tm` arcs (2 when no row of the graph has more than two, which is every
//     left-to-right chain; else 4) in registers for the whole time loop.  A row of up to tm arcs takes one lane, a
//     longer one the smallest power of two of neighbouring lanes that holds it (the kernel combines them when the
//     slice's sums are formed); all rows of a slice take the same number of lanes.
//   * Every state is a row, also one without arcs (all its arcs weigh zero-bar): the kernel needs no list of such rows,
//     and writing every state at every step keeps both buffers right.
//   * Rows are sorted by the lanes they take, widest first, and keep their order otherwise; slice s goes to wave
//     s mod NC of the workgroup.
#include <algorithm>
#include <cmath>

#include "fb_internal.h"

namespace fb {

bool small_append(SmallHost &S, int32_t k0, int32_t K, const int64_t *ptr, const int32_t *col, const float *w)
{
    if (K > kSmallStates) return false;
    const int32_t tm = S.tm;
    // rows by the lanes they take, widest first, in ascending order otherwise (a counting sort)
    std::vector<int32_t> order((size_t)K);
    std::vector<int8_t> lg_of((size_t)K);
    int32_t at_lg[8] = {0};
    for (int32_t r = 0; r < K; ++r) {
        const int64_t n = ptr[r + 1] - ptr[r];
        int lg = 0;
        while (lg <= 6 && n > ((int64_t)tm << lg)) ++lg;
        if (lg > 6) return false;
        lg_of[(size_t)r] = (int8_t)lg;
        ++at_lg[6 - lg + 1];
    }
    for (int i = 1; i < 8; ++i) at_lg[i] += at_lg[i - 1];
    for (int32_t r = 0; r < K; ++r) order[(size_t)at_lg[6 - lg_of[(size_t)r]]++] = r;
    SmallSub sd{};
    sd.k0 = k0;
    sd.K = K;
    sd.slice0 = (int32_t)S.lg.size();
    int at = kWave, lg_slice = 0;   // lanes used of the slice being filled
    for (const int32_t r : order) {
        const int lg = lg_of[(size_t)r];
        if (at >= kWave) {   // (a row that needs fewer lanes than its slice gives takes them all the same)
            lg_slice = lg;
            S.lg.push_back(lg);
            S.rows.resize(S.rows.size() + kWave, kSmallNoRow);
            S.arcs.resize(S.arcs.size() + (size_t)tm * kWave, Arc{0, -INFINITY});
            at = 0;
        }
        const size_t slice = S.lg.size() - 1;
        S.rows[slice * kWave + (size_t)at] = (uint32_t)r;
        const int64_t n = ptr[r + 1] - ptr[r];
        Arc *a = S.arcs.data() + slice * (size_t)tm * kWave + (size_t)at;
        for (int64_t i = 0; i < n; ++i) {
            const int64_t e = ptr[r] + i;
            a[(size_t)(i % tm) * kWave + (size_t)(i / tm)] = Arc{col[e] * 8, w[e]};
        }
        at += 1 << lg_slice;
    }
    sd.n_slice = (int32_t)S.lg.size() - sd.slice0;
    if (sd.n_slice > kSmallMaxSlices) return false;
    S.max_slices = std::max(S.max_slices, sd.n_slice);
    S.sub.push_back(sd);
    return true;
}

// Every index the kernel forms stays inside what it indexes.
bool small_in_bounds(const SmallHost &S, std::string &why)
{
    const size_t n = S.lg.size();
    if (S.rows.size() != n * kWave || S.arcs.size() != n * (size_t)S.tm * kWave || (S.tm != 2 && S.tm != 4)) { why = "small plan: sizes"; return false; }
    for (const SmallSub &sd : S.sub) {
        if (sd.slice0 < 0 || sd.n_slice < 1 || (size_t)sd.slice0 + (size_t)sd.n_slice > n || sd.K < 1 || sd.K > kSmallStates) { why = "small plan: sub-graph"; return false; }
        std::vector<char> seen((size_t)sd.K, 0);
        for (int32_t s = sd.slice0; s < sd.slice0 + sd.n_slice; ++s) {
            if (S.lg[(size_t)s] < 0 || S.lg[(size_t)s] > 6 || (S.tm == 2 && S.lg[(size_t)s] != 0)) { why = "small plan: lanes per row"; return false; }
            for (int lane = 0; lane < kWave; ++lane) {
                const uint32_t r = S.rows[(size_t)s * kWave + lane];
                if (r != kSmallNoRow) {
                    if (r >= (uint32_t)sd.K || seen[r]) { why = "small plan: row"; return false; }
                    seen[r] = 1;
                }
                for (int t = 0; t < S.tm; ++t) {
                    const Arc &a = S.arcs[((size_t)s * S.tm + t) * kWave + lane];
                    if (a.src < 0 || a.src % 8 || a.src / 8 >= sd.K || std::isnan(a.w)) { why = "small plan: arc"; return false; }
                }
            }
        }
        for (const char c : seen)
            if (!c) { why = "small plan: a state without a row"; return false; }
    }
    return true;
}

// Whether the vectors of a graph's recursions keep within a double's range (fb_small_linear.hip).  Mass that lies far behind the
// frame's largest entry comes from states that get theirs from elsewhere and pass it on over many steps, or that nobody refreshes: a
// cycle beside the main one whose states decay (or are left behind) by some binary orders every frame.  So: finite weights of
// ordinary size, one cycle-bearing component, and every state on it or hanging off it within kDeep steps either way - an
// entry then lies at most kDeep arcs and emissions behind the largest (twice 24 steps of 20 nats each are 1400 of the 1100
// binary orders there are up to the largest: met by no emissions but masks, and a run that leaves the range is only slower).
// Measured, a direction in the log form -> in the probability domain, us: 701 states, 3.5 k arcs, 97 pdfs, 23 x 211 frames 253 -> 130
// (300 pdfs 259 -> 156); 1000 states, 4 k arcs, 16 x 200 242 -> 135; 300 states, 1.2 k arcs, 8 x 200 131 -> 62; 120 states 97 -> 68; 60
// states 80 -> 47; 30 states 65 -> 38.
bool small_mixes(int32_t K, const std::vector<int64_t> &in_ptr, const std::vector<int32_t> &in_src, const std::vector<float> &in_w,
                 const std::vector<int64_t> &out_ptr, const std::vector<int32_t> &out_dst, const std::vector<float> &out_w,
                 const std::vector<float> &init2, const std::vector<float> &final2)
{
    constexpr int kDeep = 24;
    constexpr float kNone = -1.0e30f, kLow = -100.0f, kHigh = 40.0f;
    auto ordinary = [&](float x) { return x <= kNone || (x >= kLow && x <= kHigh); };   // (false for a NaN)
    auto rows_ok = [&](const std::vector<int64_t> &ptr, const std::vector<float> &w) {
        for (int32_t r = 0; r < K; ++r) {
            float top = kNone;
            for (int64_t i = ptr[(size_t)r]; i < ptr[(size_t)r + 1]; ++i) {
                if (!ordinary(w[(size_t)i])) return false;
                top = std::max(top, w[(size_t)i]);
            }
            // (a sum of n weights is at most n times the largest)
            if (top > kNone && (double)top + std::log2((double)(ptr[(size_t)r + 1] - ptr[(size_t)r])) > (double)kHigh) return false;
        }
        return true;
    };
    if (!rows_ok(in_ptr, in_w) || !rows_ok(out_ptr, out_w)) return false;
    for (int32_t k = 0; k < K; ++k)
        if (!ordinary(init2[(size_t)k]) || !ordinary(final2[(size_t)k])) return false;

    // steps from `from` to every state it reaches (-1: none) along the arcs of rows
    auto steps = [&](int32_t from, const std::vector<int64_t> &ptr, const std::vector<int32_t> &to, const std::vector<float> &w) {
        std::vector<int32_t> d((size_t)K, -1), queue{from};
        d[(size_t)from] = 0;
        for (size_t h = 0; h < queue.size(); ++h)
            for (int64_t i = ptr[(size_t)queue[h]]; i < ptr[(size_t)queue[h] + 1]; ++i) {
                const int32_t t = to[(size_t)i];
                if (w[(size_t)i] > kNone && d[(size_t)t] < 0) {
                    d[(size_t)t] = d[(size_t)queue[h]] + 1;
                    queue.push_back(t);
                }
            }
        return d;
    };
    // what is left when states without an arc in (or out) from what is left are taken away again and again holds all cycles,
    // and is the one component if its states all reach each other
    std::vector<char> left((size_t)K, 1);
    std::vector<int32_t> n_in((size_t)K, 0), n_out((size_t)K, 0), gone;
    for (int32_t r = 0; r < K; ++r)
        for (int64_t i = out_ptr[(size_t)r]; i < out_ptr[(size_t)r + 1]; ++i)
            if (out_w[(size_t)i] > kNone) { ++n_out[(size_t)r]; ++n_in[(size_t)out_dst[(size_t)i]]; }
    for (int32_t k = 0; k < K; ++k)
        if (n_in[(size_t)k] == 0 || n_out[(size_t)k] == 0) { left[(size_t)k] = 0; gone.push_back(k); }
    while (!gone.empty()) {
        const int32_t k = gone.back();
        gone.pop_back();
        auto take = [&](const std::vector<int64_t> &ptr, const std::vector<int32_t> &to, const std::vector<float> &w, std::vector<int32_t> &count) {
            for (int64_t i = ptr[(size_t)k]; i < ptr[(size_t)k + 1]; ++i) {
                const int32_t t = to[(size_t)i];
                if (w[(size_t)i] > kNone && --count[(size_t)t] == 0 && left[(size_t)t]) { left[(size_t)t] = 0; gone.push_back(t); }
            }
        };
        take(out_ptr, out_dst, out_w, n_in);
        take(in_ptr, in_src, in_w, n_out);
    }
    int32_t root = 0;
    while (root < K && !left[(size_t)root]) ++root;
    if (root == K) return false;                            // (no cycle: the mass dies after at most K frames)
    const std::vector<int32_t> from = steps(root, out_ptr, out_dst, out_w), to = steps(root, in_ptr, in_src, in_w);
    for (int32_t k = 0; k < K; ++k) {
        if (left[(size_t)k] && (from[(size_t)k] < 0 || to[(size_t)k] < 0)) return false;
        if (from[(size_t)k] > kDeep || to[(size_t)k] > kDeep) return false;
    }
    return true;
}

void small_apply_host(const SmallHost &S, int32_t sub, const double *x, double *y)
{
    const SmallSub &sd = S.sub[(size_t)sub];
    for (int32_t s = sd.slice0; s < sd.slice0 + sd.n_slice; ++s) {
        const int g = 1 << S.lg[(size_t)s];
        for (int lane = 0; lane < kWave; lane += g) {
            const uint32_t r = S.rows[(size_t)s * kWave + lane];
            if (r == kSmallNoRow) continue;
            double m = -INFINITY, acc = 0.0;
            for (int pass = 0; pass < 2; ++pass)
                for (int l = lane; l < lane + g; ++l)
                    for (int t = 0; t < S.tm; ++t) {
                        const Arc &a = S.arcs[((size_t)s * S.tm + t) * kWave + l];
                        const double v = (double)a.w + x[a.src / 8];
                        if (pass == 0) m = std::max(m, v);
                        else if (m > -INFINITY) acc += std::exp2(v - m);
                    }
            y[r] = m > -INFINITY ? m + std::log2(acc) : m;
        }
    }
}

}  // namespace fb
