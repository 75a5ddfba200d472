"""The probability-domain recursion at the sizes where its data-moving wave and its emission rows can go wrong: rows of
emissions that end at, just below and just behind a wave-wide piece and that may or may not be read in 16-byte pieces,
rows of states of every remainder, waves with more units than stay in registers, runs of one to a few frames.  Against
the oracle; tolerances as elsewhere: log Z 1e-4 relative, posteriors 1e-5."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


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


def test_rows_of_a_stream_of_frames_stay_what_they_were():
    """Rows leave by 16-byte stores whose registers are used again at once: three calls give the same bytes, and the same
    as a batch of one gives."""
    import torch

    import paper_2112_00709_amd as fb
    rng = np.random.default_rng(8)
    D = 84
    den = wl.random_graph(rng, 2303, D, mean_extra_deg=14.0)
    emis = (rng.standard_normal((8, 60, D)) * 2).astype(np.float32)
    e, l = torch.from_numpy(emis).cuda(), torch.full((8,), 60, dtype=torch.int32).cuda()
    G = fb.graph_from(den, D)
    for call in (fb.fb_alpha, fb.fb_beta):
        first = call(G, e, l)[0].clone()
        for _ in range(2):
            assert torch.equal(call(G, e, l)[0], first)
        for q in (0, 7):
            one = call(G, e[q:q + 1].contiguous(), l[q:q + 1])[0]
            assert torch.equal(one[0], first[q])
    G.destroy()
