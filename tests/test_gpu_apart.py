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


def _check(fb, g, D, emis, lengths, rows=None):
    """alpha, beta, posteriors against the oracle; the restarts of fb_alpha."""
    import torch
    h = fb.graph_from(g, D)
    assert fb.fb_graph_linear_weights(h) == 2
    before = fb.fb_debug_linear_restarts()
    fb.fb_alpha(h, torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda())
    given_up = fb.fb_debug_linear_restarts() - before
    h.destroy()
    compare_fb(fb, g, D, emis, lengths, sel=list(range(lengths.size)) if rows is None else rows, name="states apart")
    return given_up


@pytest.mark.parametrize("K,D,deg,T", [(1100, 40, 2, 37), (1300, 64, 5, 12), (3001, 90, 13, 23)])
def test_every_step_may_be_the_one_that_takes_them_out(fb, K, D, deg, T):
    """The states apart fall out of a float's range at one frame, another for every sequence, the last among them; no call is too
    short.  (Of the first two frames the run is done over in the log form: the step before is not there to go back to.)"""
    rng = np.random.default_rng(K)
    g = _graph(rng, K, D, deg, 3)
    emis = (rng.standard_normal((T + 1, T, D)) * 2).astype(np.float32)
    for f in range(T):
        emis[f, f, D - 1] = -300.0
    lengths = np.full(T + 1, T, dtype=np.int32)
    lengths[5] = 6                                           # (the last frame of a shorter sequence)
    assert _check(fb, g, D, emis, lengths) == 2


def test_states_that_stay_in_range_stay_in_the_plan(fb):
    """As fast as they were before they could run apart: the same launch over a graph with such states and one without."""
    import torch
    rng = np.random.default_rng(7)
    D, T, B = 60, 100, 64
    graphs = [_graph(rng, 1500, D, 2.5, 2)]
    graphs[0].logw[(graphs[0].src >= 1500) & (graphs[0].dst >= 1500)] = -1.0
    graphs.append(wl.Graph(**{**graphs[0].__dict__}))
    graphs[1].src, graphs[1].dst = np.append(graphs[1].src, np.full(6, 11, np.int32)), np.append(graphs[1].dst, np.arange(1500, 1506, dtype=np.int32))
    graphs[1].logw = np.append(graphs[1].logw, np.full(6, -1.0, np.float32))   # (an arc from the rest into every one of them)
    emis = torch.from_numpy((rng.standard_normal((B, T, D)) * 0.5).astype(np.float32)).cuda()
    emis[:, :, D - 1] = 1.7                                  # (the rest gains ln(1.75) a frame, the cycle loses some 1)
    l = torch.full((B,), T, dtype=torch.int32, device="cuda")
    times = []
    for g in graphs:
        h = fb.graph_from(g, D)
        best = np.inf
        before = fb.fb_debug_linear_restarts()
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                fb.fb_alpha(h, emis, l)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 100.0)
        assert fb.fb_debug_linear_restarts() == before
        times.append(best)
        h.destroy()
    print(f"[gpu-case] in range: {times[0]:.1f} us, no states apart: {times[1]:.1f} us", flush=True)
    assert times[0] <= 1.2 * times[1]                        # (apart from the first step on: 1.5)


@pytest.mark.parametrize("kind", ["-inf", "mask", "mask all", "-inf all"])
def test_unusual_emissions(fb, kind):
    """Of the states apart, or of all, in a frame while they are in the plan (frame 4) and one in which they run apart (frame 30)."""
    rng = np.random.default_rng(len(kind))
    D, T = 50, 44
    g = _graph(rng, 1300, D, 4, 3)
    emis = (rng.standard_normal((3, T, D)) * 2).astype(np.float32)
    emis[:, 12, D - 1] = -200.0
    value = -np.inf if "inf" in kind else -1.0e20
    at = slice(None) if "all" in kind else D - 1
    emis[0, 4, at] = value
    emis[1, 30, at] = value
    lengths = np.full(3, T, dtype=np.int32)
    if "all" in kind:                                        # (log Z is the mask's, or there is no path: checked as such)
        import torch
        h = fb.graph_from(g, D)
        e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
        a, _, za = fb.fb_alpha(h, e, l)
        b, _, zb = fb.fb_beta(h, e, l)
        gam, _ = fb.fb_posteriors(h, a, b, l, 3, T)
        ref = oracle.forward_backward(g, emis, lengths)
        for z in (za.cpu().numpy(), zb.cpu().numpy()):
            assert np.all(np.isneginf(z) == np.isneginf(ref.logz))
            fin = np.isfinite(ref.logz)
            assert np.all(np.abs(z[fin] - ref.logz[fin]) <= 1e-4 * np.abs(ref.logz[fin]))
        assert np.abs(gam[2].cpu().numpy() - ref.gamma[2]).max() <= 1e-5
        h.destroy()
    else:
        assert _check(fb, g, D, emis, lengths) == 0


def test_a_nan_stays_one(fb):
    import torch
    rng = np.random.default_rng(5)
    D, T = 50, 40
    g = _graph(rng, 1300, D, 4, 3)
    emis = (rng.standard_normal((4, T, D)) * 2).astype(np.float32)
    emis[2:, 12, D - 1] = -300.0
    emis[0, 20, D - 1] = np.nan                              # of a state apart in the plan, of one of the rest, and either when they run apart
    emis[1, 20, int(g.pdf[7])] = np.nan
    emis[3, 20, int(g.pdf[7])] = np.nan
    h = fb.graph_from(g, D)
    a, _, z = fb.fb_alpha(h, torch.from_numpy(emis).cuda(), torch.full((4,), T, dtype=torch.int32, device="cuda"))
    z = z.cpu().numpy()
    assert np.isnan(z[[0, 1, 3]]).all() and np.isfinite(z[2])
    assert np.isnan(a[0, T - 1].cpu().numpy()).any()
    h.destroy()


@pytest.mark.parametrize("what,taken", [("64 states", True), ("65 states", False), ("4 arcs", True), ("5 arcs", False), ("cloned target", True)])
def test_what_may_run_apart(fb, what, taken):
    """The limits, from both sides; a state of the rest whose row is spread over clones and takes arcs of theirs."""
    rng = np.random.default_rng(len(what) + ord(what[0]))
    D, T = 50, 30
    K = 2300 if what == "cloned target" else 1300
    g = _graph(rng, K, D, 2 if K > 2000 else 4, {"64 states": 61, "65 states": 62}.get(what, 6))   # (drain is not among them: it neither lasts nor feeds one that does)
    if "arcs" in what:                                       # (the fed state gets an arc from the first and one from the last of the cycle)
        n = int(what[0]) - 2
        g.src, g.dst = np.append(g.src, K + np.arange(1, 1 + n)).astype(np.int32), np.append(g.dst, np.full(n, K + 6)).astype(np.int32)
        g.logw = np.append(g.logw, np.full(n, -1.0)).astype(np.float32)
        assert np.unique(g.src[g.dst == K + 6]).size == int(what[0])
    if what == "cloned target":
        every = np.arange(K, dtype=np.int32)
        g.src, g.dst = np.concatenate([g.src, every, [K, K + 1]]).astype(np.int32), np.concatenate([g.dst, np.full(K + 2, 9)]).astype(np.int32)
        g.logw = np.concatenate([g.logw, -rng.exponential(size=K + 2)]).astype(np.float32)
    emis = (rng.standard_normal((2, T, D)) * 2).astype(np.float32)
    emis[:, 9, D - 1] = -300.0
    assert _check(fb, g, D, emis, np.full(2, T, dtype=np.int32)) == (0 if taken else 2)


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
