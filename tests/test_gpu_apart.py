"""Large shared graphs with states that get nothing from the rest of the graph: run apart inside the probability-domain
kernel while they fall behind, lead, or both are so close that a float holds them; redone in the log form where they come to matter again
after a float has lost them."""
import numpy as np
import pytest

import oracle
import paper_2112_00709_amd as fb_module
import workloads as wl
from test_gpu_parity import compare_fb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    return fb_module


def _graph(rng, K, D, deg, n_cycle, final_main=True):
    """A mixing graph of K states and, behind them, a cycle of n_cycle states that nothing enters, a state only it feeds, one
    that feeds it and has no arc in (and feeds another that nothing else enters), and a state with a self-loop; all have arcs into the rest.  Their pdf is D - 1, nobody else's."""
    n = int(K * deg)
    src, dst = np.concatenate([np.arange(K), rng.integers(0, K, n)]), np.concatenate([(np.arange(K) + 1) % K, rng.integers(0, K, n)])
    cyc = K + np.arange(n_cycle)
    fed, feeds, loop, drain = K + n_cycle, K + n_cycle + 1, K + n_cycle + 2, K + n_cycle + 3
    extra = [(c, K + (c - K + 1) % n_cycle) for c in cyc] + [(cyc[0], fed), (cyc[-1], fed), (feeds, cyc[0]), (loop, loop), (feeds, 3), (feeds, drain), (drain, 5)]
    extra += [(s, int(rng.integers(0, K))) for s in list(cyc) * 3 + [fed, fed, loop]]
    src = np.concatenate([src, [a for a, _ in extra]]).astype(np.int32)
    dst = np.concatenate([dst, [b for _, b in extra]]).astype(np.int32)
    total = K + n_cycle + 4
    pdf = rng.integers(0, D - 1, total).astype(np.int32)
    pdf[K:] = D - 1
    final = np.zeros(total, np.float32)
    if not final_main:
        final[:K] = -np.inf
    return wl.Graph(total, src, dst, (-rng.exponential(size=src.size)).astype(np.float32), pdf, np.full(total, -np.log(total), np.float32), final)


def _emissions(rng, D, T):
    """Five courses of the pdf of the states apart: far behind, close, ahead, lost and then ahead, ahead and then lost."""
    emis = (rng.standard_normal((5, T, D)) * 2).astype(np.float32)
    emis[0, :, D - 1] = -12.0
    emis[2, :, D - 1] = 9.0
    emis[3, :16, D - 1] = -12.0                              # (some 220 nats: more than a float's range, not so much that the log form rounds at 1e-4)
    emis[3, 16:, D - 1] = 12.0
    emis[4, : T // 4, D - 1] = 7.0
    emis[4, T // 4:, D - 1] = -12.0
    return emis


@pytest.mark.parametrize("K,D,deg,n_cycle", [(1100, 40, 2, 1), (1300, 101, 4, 2), (3001, 90, 13, 7), (1500, 64, 3, 60)])
def test_alpha_beta_posteriors(fb, K, D, deg, n_cycle):
    import torch
    rng = np.random.default_rng(K)
    g = _graph(rng, K, D, deg, n_cycle)
    h = fb.graph_from(g, D)
    assert fb.fb_graph_linear_weights(h) == 2
    T = 70
    lengths = np.array([T, T, T - 1, T, T], dtype=np.int32)
    emis = _emissions(rng, D, T)
    before = fb.fb_debug_linear_restarts()
    fb.fb_alpha(h, torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda())
    assert fb.fb_debug_linear_restarts() - before == 1       # the fourth sequence
    h.destroy()
    out = compare_fb(fb, g, D, emis, lengths, sel=[0, 1, 2, 4], name=f"states apart, K={K}")
    # (the fourth's rows are the log form's, floats some 220 below their row's largest: log Z, and posteriors to such floats' rounding)
    ref = oracle.forward_backward(g, emis, lengths, sel=[3])
    assert abs(out["logz"][3] - ref.logz[0]) <= 1e-4 * abs(ref.logz[0]) and abs(out["logz_b"][3] - ref.logz[0]) <= 1e-4 * abs(ref.logz[0])
    tol = 1e-5 + 2.0 ** -24 * 2 * 300
    assert np.abs(out["gamma"][3] - ref.gamma[0]).max() <= tol and np.abs(out["rho"][3] - ref.rho[0]).max() <= tol


def test_log_z_of_lost_states(fb):
    """Only the states apart may end a sequence: log Z is theirs, which a float has lost."""
    import torch
    rng = np.random.default_rng(8)
    g = _graph(rng, 1300, 50, 4, 3, final_main=False)
    emis = _emissions(rng, 50, 66)
    before = fb.fb_debug_linear_restarts()
    h = fb.graph_from(g, 50)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(np.full(5, 66, np.int32)).cuda()
    z = fb.fb_alpha(h, e, l)[2].cpu().numpy()
    assert fb.fb_debug_linear_restarts() - before >= 2       # (the first and the last, which end with those states lost)
    want = oracle.forward_backward(g, emis, np.full(5, 66, np.int32)).logz
    assert np.all(np.abs(z - want) <= 1e-4 * np.abs(want))
    h.destroy()


def test_objective_and_gradient(fb):
    import torch
    rng = np.random.default_rng(9)
    D, T = 60, 70
    den = _graph(rng, 1300, D, 4, 5)
    phones = np.array([6, 7, 5, 8, 6])
    num = wl.chain_graphs(rng, phones, D)
    lengths = np.array([T, T - 3, T, T, T - 1], dtype=np.int32)
    emis = _emissions(rng, D, T)
    hd, hn = fb.graph_from(den, D), fb.graph_from(num, D)
    before = fb.fb_debug_linear_restarts()
    loss, zn, zd, grad = fb.lfmmi_loss_grad(hd, hn, torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda())
    # (of ten runs: the forward one of the fourth sequence, and backward ones in which those states lead for good)
    assert 1 <= fb.fb_debug_linear_restarts() - before <= 5
    ref = oracle.lfmmi(den, num, emis, lengths)
    zn, zd, grad = zn.cpu().numpy(), zd.cpu().numpy(), grad.cpu().numpy()
    assert np.all(np.abs(zd - ref.logz_den) <= 1e-4 * np.abs(ref.logz_den)) and np.all(np.abs(zn - ref.logz_num) <= 1e-4 * np.abs(ref.logz_num))
    for b in range(5):
        tol = 1e-5 + (2.0 ** -24 * 2 * 300 if b == 3 else 0.0)   # (see above)
        assert np.abs(grad[b, :lengths[b]] - ref.grad[b][:lengths[b]]).max() <= tol
    hd.destroy(); hn.destroy()
