"""The probability-domain recursion at the sizes where its data-moving wave and its emission rows can go wrong: rows of
emissions that end at, just below and just behind a wave-wide piece and that may or may not be read in 16-byte pieces,
rows of states of every remainder, waves with more units than stay in registers, runs of one to a few frames.  Against
the oracle; tolerances as elsewhere: log Z 1e-4 relative, posteriors 1e-5."""
import numpy as np
import pytest

import oracle
import workloads as wl
from oracle import leaky as oleaky

pytestmark = pytest.mark.gpu


def _rows_agree(rows, shifts, want, lengths):
    for x, c, w, T in zip(rows, shifts, want, lengths):
        x, c, w = x[:T], c[:T], w[:T]
        assert np.array_equal(np.isneginf(x), np.isneginf(w))
        fin = np.isfinite(w)
        assert np.all(np.abs((x + c[:, None])[fin] - w[fin]) <= 1e-4 * np.maximum(1.0, np.abs(w[fin])))


@pytest.mark.parametrize("K,deg,zipf,D", [(1028, 3.0, None, 252), (1025, 3.0, None, 253), (1026, 3.0, None, 254), (1027, 3.0, None, 255),
                                          (1279, 2.0, 1.1, 256), (1281, 2.0, None, 257), (1536, 7.0, 1.1, 511), (2047, 4.0, None, 1021),
                                          (2305, 15.0, None, 2047), (5999, 9.0, None, 510), (6001, 9.0, 1.1, 3001), (1100, 3.0, None, 3560)])
def test_emission_rows_and_rows_of_states(K, deg, zipf, D):
    import torch

    import paper_2112_00709_amd as fb
    rng = np.random.default_rng(K + D)
    den = wl.random_graph(rng, K, D, mean_extra_deg=deg, zipf_s=zipf)
    lengths = np.array([5, 1, 2, 3, 12, 4], dtype=np.int32)
    N = 12
    emis = (rng.standard_normal((6, N, D)) * 2).astype(np.float32)
    emis[2, 1, : D // 2] = -np.inf          # pdfs that a frame rules out: the run may leave its range and be done over
    ref = oracle.forward_backward(den, emis, lengths)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    G = fb.graph_from(den, D)
    assert fb.fb_graph_linear_weights(G) == 2
    a, ca, za = fb.fb_alpha(G, e, l)
    b, cb, zb = fb.fb_beta(G, e, l)
    _, rho = fb.fb_posteriors(G, a, b, l, 6, N, want_state=False)
    torch.cuda.synchronize()
    a, ca, b, cb, za, zb, rho = (t.cpu().numpy() for t in (a, ca, b, cb, za, zb, rho))
    for q, T in enumerate(lengths):
        for z in (za[q], zb[q]):
            assert abs(z - ref.logz[q]) <= 1e-4 * max(1.0, abs(ref.logz[q]))
        assert np.abs(rho[q] - ref.rho[q]).max() <= 1e-5
        for x, c, want in ((a[q, :T], ca[q, :T], ref.alpha[q]), (b[q, :T], cb[q, :T], ref.beta[q])):
            assert np.array_equal(np.isneginf(x), np.isneginf(want[:T]))
            fin = np.isfinite(want[:T])
            assert np.all(np.abs((x + c[:, None])[fin] - want[:T][fin]) <= 1e-4 * np.maximum(1.0, np.abs(want[:T][fin])))
    G.destroy()


@pytest.mark.parametrize("K,deg", [(2500, 9.0), (3003, 9.6), (2303, 14.0), (3500, 13.0)])
def test_rows_of_a_stream_of_frames_stay_what_they_were(K, deg):
    """Rows leave by 16-byte stores whose registers are used again at once: they are the oracle's, three calls give the same
    bytes, and a batch of one gives the same.  The kernels of up to 16 and up to 20 units a wave and, twice, the general one;
    rows of whole groups of eight pieces, with and without a partial group behind them."""
    import torch

    import paper_2112_00709_amd as fb
    rng = np.random.default_rng(8)
    D = 84
    den = wl.random_graph(rng, K, D, mean_extra_deg=deg)
    emis = (rng.standard_normal((8, 60, D)) * 2).astype(np.float32)
    lengths = np.full(8, 60, dtype=np.int32)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    ref = oracle.forward_backward(den, emis, lengths)
    G = fb.graph_from(den, D)
    for call, want in ((fb.fb_alpha, ref.alpha), (fb.fb_beta, ref.beta)):
        first, shift, _ = call(G, e, l)
        first = first.clone()
        _rows_agree(first.cpu().numpy(), shift.cpu().numpy(), want, lengths)
        for _ in range(2):
            assert torch.equal(call(G, e, l)[0], first)
        for q in (0, 7):
            one = call(G, e[q:q + 1].contiguous(), l[q:q + 1])[0]
            assert torch.equal(one[0], first[q])
    G.destroy()


@pytest.mark.parametrize("K,deg", [(1200, 3.0), (3003, 9.6), (3000, 15.0)])
def test_vectors_that_fall_too_far_in_one_step(K, deg):
    """A pdf that no state has lies 124.5 binary orders above the rest in one frame, and in the frames beside it one state
    holds nearly all the mass, with arcs of weight 1/16: the vector falls by more than 126 binary orders in that step, so
    that its scale for the next would not be a float, although no emission's factor is too small for one and every entry
    stays above the smallest allowed.  Such a run is done over in the log form.  The frame is in the middle, next to either
    end (the last step that a run can be stopped for), and the first or the last (not stopped: a first vector
    has a scale of its own, the last one needs none, and log Z is taken from it).  Rows as logarithms, rows as kept, the
    leaky mode."""
    import torch

    import paper_2112_00709_amd as fb
    rng = np.random.default_rng(K)
    D = 60
    den = wl.random_graph(rng, K, D, mean_extra_deg=deg)
    den.pdf[:] = den.pdf % (D - 2)
    hub = int(np.argmax(np.minimum(np.bincount(den.src, minlength=K), np.bincount(den.dst, minlength=K))))
    den.pdf[hub] = D - 2
    den.logw[(den.src == hub) | (den.dst == hub)] = np.log(1 / 16)
    lengths = np.array([12, 12, 12, 11, 12, 12, 3, 2], dtype=np.int32)
    far = [None, 5, 10, 1, 11, 0, 1, None]
    B, N = len(far), 12
    num = wl.chain_graphs(rng, np.maximum(1, lengths // 4), D)
    num.pdf[:] = num.pdf % (D - 2)
    emis = (rng.standard_normal((B, N, D)) * 2).astype(np.float32)
    for b, f in enumerate(far):
        if f is not None:
            emis[b, f] = rng.standard_normal(D) * 0.05
            emis[b, f, D - 1] = 124.5 * np.log(2)
            for q in (f - 1, f + 1):
                if 0 <= q < lengths[b]:
                    emis[b, q] = rng.standard_normal(D) * 0.05
                    emis[b, q, D - 2] = 20.0
    over = sum(f is not None and 1 <= f <= T - 2 for f, T in zip(far, lengths))
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    ref = oracle.forward_backward(den, emis, lengths)
    lf = oracle.lfmmi(den, num, emis, lengths)
    leaky = oleaky.forward_backward(den, emis, lengths, 1e-3)
    G, H = fb.graph_from(den, D), fb.graph_from(num, D)
    assert fb.fb_graph_linear_weights(G) == 2
    count = [fb.fb_debug_linear_restarts()]

    def restarts():
        torch.cuda.synchronize()
        count.append(fb.fb_debug_linear_restarts())
        return count[-1] - count[-2]

    a, ca, za = fb.fb_alpha(G, e, l)
    assert restarts() == over
    b_, cb, zb = fb.fb_beta(G, e, l)
    assert restarts() == over
    _, rho = fb.fb_posteriors(G, a, b_, l, B, N, want_state=False)
    _, _, zd, grad = fb.lfmmi_loss_grad(G, H, e, l)
    assert restarts() == 2 * over
    zl, post = fb.fb_leaky_posteriors(G, e, l, 1e-3)
    torch.cuda.synchronize()
    a, ca, b_, cb, rho, grad, post = (t.cpu().numpy() for t in (a, ca, b_, cb, rho, grad, post))
    for name, z, want in (("alpha", za, ref.logz), ("beta", zb, ref.logz), ("lfmmi", zd, ref.logz), ("leaky", zl, leaky.logz)):
        assert np.all(np.abs(z.cpu().numpy() - want) <= 1e-4 * np.maximum(1.0, np.abs(want))), (name, z.cpu().numpy() - want)
    _rows_agree(a, ca, ref.alpha, lengths)
    _rows_agree(b_, cb, ref.beta, lengths)
    for x, want in ((rho, ref.rho), (grad, lf.grad), (post, leaky.rho)):
        assert np.abs(x - want).max() <= 1e-5
    G.destroy(); H.destroy()
