"""The small-graph recursion on probabilities at the sizes where it can go wrong: around what its variants hold (states,
slices, pdfs per lane), rows over one to 64 lanes, sequences shorter than the rounds of its waves, and runs that leave
the range or meet masks, which the log form does over."""
import numpy as np
import pytest

import oracle
import paper_2112_00709_amd as fb
import workloads as wl
from test_gpu_small_graphs import _check

pytestmark = pytest.mark.gpu


def _graph(rng, K, deg, hub, D):
    """One strongly connected part: a cycle through every state but the last two, which hang off it (one without an arc in)."""
    n = int(K * deg)
    core = max(1, K - 2)
    src, dst = rng.integers(0, core, n), rng.integers(0, core, n)
    order = rng.permutation(core)
    for lead in (1, 7):                                      # (a cycle, and a shorter way round it)
        src, dst = np.concatenate([src, order]), np.concatenate([dst, np.roll(order, -lead)])
    src, dst = np.concatenate([src, np.arange(hub) % core, np.full(hub, core - 1)]), np.concatenate([dst, np.full(hub, core // 3), np.arange(hub) % core])
    if K > 2:
        src, dst = np.concatenate([src, [K - 2, 0, 0]]), np.concatenate([dst, [0, K - 1, K - 1]])
    logw = (-rng.exponential(size=src.size)).astype(np.float32)
    init = (-rng.exponential(size=K)).astype(np.float32)
    init[rng.integers(0, K)] = -np.inf
    return wl.Graph(K, src.astype(np.int32), dst.astype(np.int32), logw, rng.integers(0, D, K).astype(np.int32), init if K > 1 else init * 0,
                    (-rng.exponential(size=K)).astype(np.float32))


SIZES = [(4, 3, 0, 3, (1, 2, 3, 4)), (16, 2, 6, 16, (5, 7, 8, 9)), (30, 3, 0, 40, (15, 16, 17, 24)), (63, 1.5, 60, 5, (1, 8, 25, 33)),
         (64, 0.5, 0, 70, (31, 32, 34, 40)), (100, 1.5, 90, 128, (2, 9, 10, 11)), (128, 2, 0, 129, (6, 12, 13, 48)), (250, 1.5, 240, 130, (14, 18, 19, 20)),
         (257, 4, 100, 300, (21, 22, 23, 3)), (500, 3, 64, 512, (1, 3, 4, 5)), (513, 3, 200, 600, (6, 7, 8, 26)), (700, 2.5, 100, 97, (2, 27, 28, 29)),
         (769, 2, 33, 320, (9, 10, 11, 12)), (900, 2, 40, 321, (13, 14, 15, 16)), (1024, 1.2, 120, 1500, (4, 5, 6, 35))]


@pytest.mark.parametrize("K,deg,hub,D,frames", SIZES)
def test_parity(K, deg, hub, D, frames):
    rng = np.random.default_rng(K)
    g = _graph(rng, K, deg, hub, D)
    lengths = np.array(list(frames) + [0], dtype=np.int32)
    emis = (rng.standard_normal((lengths.size, int(lengths.max()) + 1, D)) * 2).astype(np.float32)
    for b in range(lengths.size):
        emis[b, lengths[b]:] = np.nan
    emis[1, 0, :] -= 100.0                                   # (what all pdfs of a frame share is taken off it)
    h = fb.graph_from(g, D)
    assert fb.fb_graph_small_linear(h) == 1
    h.destroy()
    before = fb.fb_debug_linear_restarts()
    _check(g, emis, lengths, D)
    assert fb.fb_debug_linear_restarts() == before


def _slices(g):
    """Slices of the larger of the two plans: rows of up to four arcs take a lane, longer ones the least power of two that holds them; widest
    rows first, a slice's lanes per row are its first row's."""
    most = 0
    for rows, cols in ((g.dst, g.src), (g.src, g.dst)):
        pairs = np.unique(rows.astype(np.int64) * g.K + cols)
        n = np.bincount(pairs // g.K, minlength=g.K)
        lanes = np.sort([1 << max(0, int(np.ceil(np.log2(max(x, 1) / 4)))) for x in n])[::-1]
        used, at, wide = 0, 64, 1
        for w in lanes:
            if at >= 64:
                used, at, wide = used + 1, 0, int(w)
            at += wide
        most = max(most, used)
    return most


def _circulant(rng, K, arcs, D):
    """Every row the same number of arcs, every pdf used where there are no more of them than states."""
    src = np.tile(np.arange(K), arcs)
    dst = (src + np.repeat(np.concatenate([[1], rng.permutation(np.arange(2, K))[:arcs - 1]]), K)) % K
    return wl.Graph(K, src.astype(np.int32), dst.astype(np.int32), (-rng.exponential(size=src.size)).astype(np.float32),
                    rng.permutation(np.arange(K) % D).astype(np.int32), (-rng.exponential(size=K)).astype(np.float32), (-rng.exponential(size=K)).astype(np.float32))


# the instantiations that SIZES does not reach: (states, arcs a row, pdfs, slices): 25 to 32 slices with up to 128, 320 and more pdfs, 17 to 24 and 9 to 16
# with as many, 5 to 8 with more than 128
LARGEST = [(455, 9, 97, 29), (455, 9, 300, 29), (455, 9, 455, 29), (810, 5, 128, 26), (511, 8, 321, 16), (400, 5, 129, 13), (220, 4, 220, 4), (130, 9, 130, 9),
           (125, 9, 129, 8), (200, 6, 200, 7)]


@pytest.mark.parametrize("K,arcs,D,slices", LARGEST)
def test_parity_of_the_largest_plans(K, arcs, D, slices):
    rng = np.random.default_rng(K + D)
    g = _circulant(rng, K, arcs, D)
    assert _slices(g) == slices and np.unique(g.pdf).size == min(D, K)
    lengths = np.array([0, 1, 2, 5, 9, 18, 33], dtype=np.int32)
    emis = (rng.standard_normal((lengths.size, int(lengths.max()) + 1, D)) * 2).astype(np.float32)
    for b in range(lengths.size):
        emis[b, lengths[b]:] = np.nan
    h = fb.graph_from(g, D)
    assert fb.fb_graph_small_linear(h) == 1
    h.destroy()
    before = fb.fb_debug_linear_restarts()
    _check(g, emis, lengths, D)
    assert fb.fb_debug_linear_restarts() == before


@pytest.mark.parametrize("K,deg,hub,D,frames", [SIZES[i] for i in (1, 3, 5, 7, 9, 11, 14)] + [(K, arcs, -1, D, None) for K, arcs, D, _ in (LARGEST[0], LARGEST[2], LARGEST[9])])
def test_runs_that_leave_the_range(K, deg, hub, D, frames):
    """Emissions hundreds of nats apart: one sequence all along, one in a single frame, one a masked state, one not at all."""
    import torch
    rng = np.random.default_rng(K)
    g = _graph(rng, K, deg, hub, D) if hub >= 0 else _circulant(rng, K, deg, D)
    T = 26
    lengths = np.array([T, T, T, T], dtype=np.int32)
    emis = (rng.standard_normal((4, T, D)) * 2).astype(np.float32)
    emis[0] *= 100.0
    emis[1, 11] *= 150.0
    emis[2, :, int(g.pdf[1])] = -1.0e4
    before = fb.fb_debug_linear_restarts()
    h = fb.graph_from(g, D)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    a, ca, za = fb.fb_alpha(h, e, l)
    b, cb, zb = fb.fb_beta(h, e, l)
    gam, rho = fb.fb_posteriors(h, a, b, l, 4, T)
    assert fb.fb_debug_linear_restarts() - before == 6       # both directions of three of them
    a, b, ca, cb, za, zb, gam, rho = (t.cpu().numpy() for t in (a, b, ca, cb, za, zb, gam, rho))
    ref = oracle.forward_backward(g, emis, lengths)
    for q in range(4):
        for z in (za[q], zb[q]):
            assert abs(z - ref.logz[q]) <= 1e-4 * max(1.0, abs(ref.logz[q]))
        tol = 1e-5 + 2.0 ** -24 * (np.abs(a[q]) + np.abs(b[q]))[ref.gamma[q] > 1e-7].max(initial=0.0)
        assert np.abs(gam[q] - ref.gamma[q]).max() <= tol and np.abs(rho[q] - ref.rho[q]).max() <= tol
        for x, c, want in ((a[q], ca[q], ref.alpha[q]), (b[q], cb[q], ref.beta[q])):
            assert np.array_equal(np.isneginf(x), np.isneginf(want))
            fin = np.isfinite(want)
            # as in _check, and the float ln 2 that shifts are multiplied by
            err = np.abs((x + c[:, None])[fin] - want[fin])
            assert np.all(err <= 1e-7 * np.abs(x[fin]) + 2e-7 * T + 1e-6 + 3e-9 * np.abs(c).max())
    h.destroy()


@pytest.mark.parametrize("K,deg,hub,D,frames", [SIZES[i] for i in (1, 4, 6, 8, 9, 11)])
@pytest.mark.parametrize("mask", [-1.0e3, -7.0e4])
def test_runs_that_end_early(K, deg, hub, D, frames, mask):
    """One pdf masked in one frame, at every place of the rounds its waves go in: the waves leave the loop together, at once or a while behind
    that frame, or at the end; so do two masks, found by different waves."""
    import torch
    rng = np.random.default_rng(K)
    g = _graph(rng, K, deg, hub, D)
    T = 41
    at = list(range(T)) + [(3, 4), (5, 11), (17, 19), (7, 40)]
    lengths = np.full(len(at) + 1, T, dtype=np.int32)
    emis = (rng.standard_normal((lengths.size, T, D)) * 2).astype(np.float32)
    for q, f in enumerate(at):
        emis[q, f, int(g.pdf[1])] = mask
    h = fb.graph_from(g, D)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    before = fb.fb_debug_linear_restarts()
    a, ca, za = fb.fb_alpha(h, e, l)
    b, cb, zb = fb.fb_beta(h, e, l)
    gam, rho = fb.fb_posteriors(h, a, b, l, lengths.size, T)
    given_up = fb.fb_debug_linear_restarts() - before
    # (of frame 0 the forward form, of the last frame the backward form may keep a mask of 1000 nats: the first vector reaches further down)
    assert 2 * len(at) - 4 <= given_up <= 2 * len(at)
    a, b, ca, cb, za, zb, gam, rho = (t.cpu().numpy() for t in (a, b, ca, cb, za, zb, gam, rho))
    ref = oracle.forward_backward(g, emis, lengths)
    for z in (za, zb):
        assert np.all(np.abs(z - ref.logz) <= 1e-6 * np.maximum(1.0, np.abs(ref.logz)))
    for q in range(lengths.size):
        # floats of the rows, as in test_runs_that_leave_the_range
        tol = 1e-5 + 2.0 ** -24 * (np.abs(a[q]) + np.abs(b[q]))[ref.gamma[q] > 1e-7].max(initial=0.0)
        assert np.abs(gam[q] - ref.gamma[q]).max() <= tol and np.abs(rho[q] - ref.rho[q]).max() <= tol
        for x, c, want in ((a[q], ca[q], ref.alpha[q]), (b[q], cb[q], ref.beta[q])):
            fin = np.isfinite(want)
            assert np.array_equal(np.isfinite(x), fin)
            assert np.all(np.abs((x + c[:, None])[fin] - want[fin]) <= 1e-7 * np.abs(x[fin]) + 2e-7 * T + 1e-6 + 3e-9 * np.abs(c).max())
    h.destroy()


@pytest.mark.parametrize("K,deg,B,taken", [(16, 3, 256, True), (16, 3, 257, False), (60, 1.5, 300, False), (150, 3, 300, True)])
def test_more_workgroups_than_compute_units(K, deg, B, taken):
    """Graphs of one computing wave go to the log form when the chip is full: nothing is given up there."""
    import torch
    rng = np.random.default_rng(K)
    D, T = 20, 6
    g = _graph(rng, K, deg, 0, D)
    h = fb.graph_from(g, D)
    assert fb.fb_graph_small_linear(h) == 1 and torch.cuda.get_device_properties(0).multi_processor_count == 256
    lengths = np.full(B, T, dtype=np.int32)
    lengths[rng.permutation(B)[:40]] = rng.integers(0, T, 40)
    emis = (rng.standard_normal((B, T, D)) * 2).astype(np.float32)
    emis[:, :, int(g.pdf[1])] = -1.0e4
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    before = fb.fb_debug_linear_restarts()
    a, _, za = fb.fb_alpha(h, e, l)
    assert fb.fb_debug_linear_restarts() - before == (np.count_nonzero(lengths) if taken else 0)
    b, _, zb = fb.fb_beta(h, e, l)
    gam, _ = fb.fb_posteriors(h, a, b, l, B, T)
    sel = np.flatnonzero(lengths)[::7]
    ref = oracle.forward_backward(g, emis, lengths, sel=sel)
    za, zb, gam = za.cpu().numpy(), zb.cpu().numpy(), gam.cpu().numpy()
    for i, q in enumerate(sel):
        for z in (za[q], zb[q]):
            assert abs(z - ref.logz[i]) <= 1e-6 * max(1.0, abs(ref.logz[i]))
        assert np.abs(gam[q][:lengths[q]] - ref.gamma[i][:lengths[q]]).max() <= 1e-5
    assert np.all(np.isneginf(za[lengths == 0]))
    h.destroy()


def _time(f):
    """us a call, the least of five rounds of ten"""
    import torch
    f()
    best = np.inf
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100.0)
    return best


@pytest.mark.parametrize("K,deg", [(40, 4), (200, 4), (701, 3)])
def test_masks_cost_no_second_run(K, deg):
    """A forbidden pdf, all along or in a late frame, costs about what it costs the log form, which the same graph with a state more that only
    keeps its own mass runs in: what is done over in that form is given up as soon as it is known, not at the end."""
    import torch
    rng = np.random.default_rng(K)
    D, T, B = 50, 200, 8
    g = _graph(rng, K, deg, 0, D)
    plus = wl.Graph(K + 1, np.append(g.src, K).astype(np.int32), np.append(g.dst, K).astype(np.int32), np.append(g.logw, -1.0).astype(np.float32),
                    np.append(g.pdf, 0).astype(np.int32), np.append(g.init, 0.0).astype(np.float32), np.append(g.final, 0.0).astype(np.float32))
    hs = [fb.graph_from(x, D) for x in (g, plus)]
    assert [fb.fb_graph_small_linear(h) for h in hs] == [1, 0]
    emis = (rng.standard_normal((B, T, D)) * 2).astype(np.float32)
    l = torch.full((B,), T, dtype=torch.int32, device="cuda")
    p = int(g.pdf[1])
    # (given up at the end as well, and slower there: 1.6 to 2.2 times; a mask of more than 65536 in the second half: 1.16 to 1.34)
    for frames, mask, most in ((slice(0, T), -1.0e4, 1.25), (slice(T // 2, T // 2 + 1), -1.0e20, 1.05)):
        x = emis.copy()
        x[:, frames, p] = mask
        e = torch.from_numpy(x).cuda()
        for f in (fb.fb_alpha, fb.fb_beta):
            t, t_log = (_time(lambda: f(h, e, l)) for h in hs)
            print(f"[gpu-case] K={K} {f.__name__} mask {mask:g}: {t:.1f} us, log form {t_log:.1f} us", flush=True)
            assert t <= most * t_log
    for h in hs:
        h.destroy()


@pytest.mark.parametrize("K,arcs", [(9, 3), (20, 4), (23, 9)])
def test_masked_frames_and_nan(K, arcs):
    """A frame of masks, one of zero-bar for all, one of zero-bar for some, a NaN: as the general kernel has them."""
    import torch
    rng = np.random.default_rng(K)
    D, T = 5, 33
    src = np.tile(np.arange(K), arcs)
    dst = (src + np.repeat(np.arange(arcs), K)) % K
    g = wl.Graph(K, src.astype(np.int32), dst.astype(np.int32), (-rng.exponential(size=src.size)).astype(np.float32),
                 rng.integers(0, D, K).astype(np.int32), np.zeros(K, np.float32), np.zeros(K, np.float32))
    h = fb.graph_from(g, D)
    assert fb.fb_graph_small_linear(h) == 1
    emis = (rng.standard_normal((5, T, D)) * 2).astype(np.float32)
    emis[0, 9] = -1e20
    emis[1, 13] = -np.inf
    emis[2, 17, 1:] = -np.inf
    emis[3, 4, int(g.pdf[0])] = np.nan
    lengths = np.full(5, T, dtype=np.int32)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    a, _, za = fb.fb_alpha(h, e, l)
    b, _, zb = fb.fb_beta(h, e, l)
    gam, _ = fb.fb_posteriors(h, a, b, l, 5, T)
    za, zb, gam = za.cpu().numpy(), zb.cpu().numpy(), gam.cpu().numpy()
    ref = oracle.forward_backward(g, emis, lengths, sel=np.array([2, 4]))
    for i, q in enumerate((2, 4)):
        both = np.isneginf(za[q]) and np.isneginf(ref.logz[i])
        assert both or (abs(za[q] - ref.logz[i]) <= 1e-4 * abs(ref.logz[i]) and abs(zb[q] - ref.logz[i]) <= 1e-4 * abs(ref.logz[i]))
        assert np.abs(gam[q] - ref.gamma[i]).max() <= 1e-5
    assert abs(za[0] / -1e20 - 1) <= 1e-6 and abs(zb[0] / -1e20 - 1) <= 1e-6 and np.isfinite(gam[0]).all()
    assert np.isneginf(za[1]) and np.isneginf(zb[1]) and np.all(gam[1] == 0)
    assert np.isnan(za[3]) and np.isnan(zb[3]) and np.isnan(gam[3]).any()
    h.destroy()
