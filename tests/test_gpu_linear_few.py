"""The probability-domain recursion where a wave's units all stay in registers: at most 16 per wave (the first four
graphs and the last) or at most 20 (the others), slices of whole pairs of units; one arc a row and rows over many lanes,
both row forms, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,deg,zipf,D", [(1025, 0.2, None, 7), (1100, 3.0, None, 40), (2000, 9.0, None, 84), (1500, 18.0, 1.1, 33),
                                          (1537, 19.0, None, 84), (3001, 8.4, None, 90), (3003, 9.6, None, 90), (5001, 0.0, None, 50)])
def test_rows_posteriors_and_gradient(K, deg, zipf, D):
    import torch

    import paper_2112_00709_amd as fb
    rng = np.random.default_rng(K)
    den = wl.random_graph(rng, K, D, mean_extra_deg=deg, zipf_s=zipf)
    lengths = np.array([11, 1, 2, 0, 16], dtype=np.int32)
    num = wl.chain_graphs(rng, np.maximum(1, lengths // 4), D)
    emis = (rng.standard_normal((5, 17, D)) * 2).astype(np.float32)
    for b, T in enumerate(lengths):
        emis[b, T:] = np.nan
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    G, H = fb.graph_from(den, D), fb.graph_from(num, D)
    assert fb.fb_graph_linear_weights(G) == 2
    fb.POISON_NEW_BUFFERS = True
    try:
        a, ca, za = fb.fb_alpha(G, e, l)
        b_, cb, zb = fb.fb_beta(G, e, l)
        _, rho = fb.fb_posteriors(G, a, b_, l, 5, 17, want_state=False)
        loss, zn, zd, grad = fb.lfmmi_loss_grad(G, H, e, l)
    finally:
        fb.POISON_NEW_BUFFERS = False
    torch.cuda.synchronize()
    a, ca, za, b_, cb, zb, rho, zd, grad = (t.cpu().numpy() for t in (a, ca, za, b_, cb, zb, rho, zd, grad))
    em = np.where(np.isnan(emis), np.float32(0), emis)
    live = np.flatnonzero(lengths > 0)
    ref = oracle.forward_backward(den, em, lengths, sel=live)
    lf = oracle.lfmmi(den, num, em, lengths, sel=live)
    for i, q in enumerate(live):
        T = int(lengths[q])
        for z in (za[q], zb[q], zd[q]):
            assert abs(z - ref.logz[i]) <= 1e-4 * max(1.0, abs(ref.logz[i]))
        assert np.abs(rho[q] - ref.rho[i]).max() <= 1e-5
        assert np.abs(grad[q] - lf.grad[i]).max() <= 1e-5
        for x, c, want in ((a[q, :T], ca[q, :T], ref.alpha[i]), (b_[q, :T], cb[q, :T], ref.beta[i])):
            assert np.array_equal(np.isneginf(x), np.isneginf(want))
            fin = np.isfinite(want)
            assert np.all(np.abs((x + c[:, None])[fin] - want[fin]) <= 1e-4 * np.maximum(1.0, np.abs(want[fin])))
    G.destroy(); H.destroy()
