"""The small-graph recursion kernel at the sizes where it can go wrong: around the states its waves hold, around its
groups of frames, rows over one to 64 lanes, rows without arcs, graphs it hands to the general kernel."""
import numpy as np
import pytest

import oracle
import paper_2112_00709_amd as fb
import workloads as wl

pytestmark = pytest.mark.gpu


def _graph(rng, K, deg, hub, D):
    """K states, about deg arcs each; `hub` arcs into one state and out of another; a state without arcs in."""
    n = int(K * deg)
    src, dst = rng.integers(0, K, n), rng.integers(0, K, n)
    dst[dst == K // 2] = 0
    src = np.concatenate([src, np.arange(K), np.arange(hub) % K, np.full(hub, K - 1)])
    dst = np.concatenate([dst, (np.arange(K) + 1) % K, np.full(hub, K // 3), np.arange(hub) % K])
    keep = dst != K // 2 if K > 3 else np.ones(dst.size, bool)
    src, dst = src[keep].astype(np.int32), dst[keep].astype(np.int32)
    logw = (-rng.exponential(size=src.size)).astype(np.float32)
    logw[rng.integers(0, logw.size, max(1, logw.size // 30))] = -np.inf
    init = (-rng.exponential(size=K)).astype(np.float32)
    init[0] = -np.inf if K > 1 else 0.0
    return wl.Graph(K, src, dst, logw, rng.integers(0, D, K).astype(np.int32), init, (-rng.exponential(size=K)).astype(np.float32))


@pytest.mark.parametrize("K,deg,hub,frames", [
    (1, 1, 0, (1, 2, 3)), (7, 2, 6, (8, 9, 10)), (64, 2, 0, (16, 17, 18)), (65, 2.2, 30, (24, 25, 33)), (128, 0.9, 0, (1, 15, 41)),
    (129, 2, 100, (7, 26, 34)), (256, 1.5, 200, (5, 6, 50)), (257, 3, 250, (12, 13, 14)), (512, 1.8, 0, (3, 31, 32)),
    (513, 2.5, 400, (19, 20, 21)), (900, 2, 256, (4, 11, 37)), (1024, 1, 100, (2, 10, 23)), (600, 2, 520, (9, 30, 31))])
def test_shared_small_graphs(K, deg, hub, frames):
    rng = np.random.default_rng(K)
    D = 11
    g = _graph(rng, K, deg, min(hub, K), D)
    lengths = np.array(list(frames) + [0], dtype=np.int32)
    B, N = lengths.size, int(lengths.max()) + 1
    emis = (rng.standard_normal((B, N, D)) * 3).astype(np.float32)
    for b in range(B):
        emis[b, lengths[b]:] = np.nan
    _check(g, emis, lengths, D)


@pytest.mark.parametrize("kind", ["chain", "ctc"])
def test_packed_small_graphs(kind):
    """One batch with sub-graphs of 3 to 1020 states: the variant is the largest one's, the others leave lanes idle."""
    D = 17
    rng = np.random.default_rng(5)
    if kind == "chain":
        phones = np.array([1, 21, 22, 43, 85, 86, 170, 171, 340])
        g = wl.chain_graphs(rng, phones, D)
        lengths = np.array([3, 66, 66, 131, 257, 259, 511, 520, 1021], dtype=np.int32)
    else:
        g = wl.ctc_graphs([rng.integers(1, D, n).tolist() for n in (1, 31, 32, 63, 64)], 0)
        lengths = np.array([1, 70, 65, 130, 140], dtype=np.int32)
    emis = (rng.standard_normal((lengths.size, int(lengths.max()), D)) * 2).astype(np.float32)
    _check(g, emis, lengths, D)


def _check(g, emis, lengths, D):
    import torch
    B, N, _ = emis.shape
    h = fb.graph_from(g, D)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    fb.POISON_NEW_BUFFERS = True
    try:
        a, ca, za = fb.fb_alpha(h, e, l)
        b, cb, zb = fb.fb_beta(h, e, l)
        gam, rho = fb.fb_posteriors(h, a, b, l, B, N)
        score, path = fb.fb_viterbi(h, e, l)
    finally:
        fb.POISON_NEW_BUFFERS = False
    torch.cuda.synchronize()
    a, b, ca, cb, za, zb, gam, rho, score, path = (t.cpu().numpy() for t in (a, b, ca, cb, za, zb, gam, rho, score, path))
    live = np.flatnonzero(lengths > 0)
    em = np.where(np.isnan(emis), np.float32(0), emis)
    ref = oracle.forward_backward(g, em, lengths, sel=live)
    best = oracle.viterbi(g, em, lengths, sel=live)
    off = g.state_off if g.packed else None
    for i, q in enumerate(live):
        T = int(lengths[q])
        rows = (lambda x: x[:T, off[q]:off[q + 1]]) if g.packed else (lambda x: x[q, :T])
        for z in (za[q], zb[q]):
            assert (np.isneginf(z) and np.isneginf(ref.logz[i])) or abs(z - ref.logz[i]) <= 1e-4 * max(1.0, abs(ref.logz[i]))
        # the rows between the calls are floats: in a long chain a state that matters lies far below its frame's best, and
        # its posterior carries half a unit of the size of its two entries
        heavy = ref.gamma[i] > 1e-7
        tol = 1e-5 + 2.0 ** -24 * (np.abs(rows(a)) + np.abs(rows(b)))[heavy].max(initial=0.0)
        assert np.abs(rows(gam) - ref.gamma[i]).max() <= tol
        assert np.abs(rho[q] - ref.rho[i]).max() <= tol
        for x, c, want in ((rows(a), ca[q, :T], ref.alpha[i]), (rows(b), cb[q, :T], ref.beta[i])):
            assert np.array_equal(np.isneginf(x), np.isneginf(want))
            fin = np.isfinite(want)
            # a stored entry is a float: half a unit of its own size, and a few units of the exponentials per frame
            err = np.abs((x + c[:, None])[fin] - want[fin])
            assert np.all(err <= 1e-7 * np.abs(x[fin]) + 2e-7 * T + 1e-6)
        if np.isneginf(best.score[i]):
            assert np.isneginf(score[q]) and np.all(path[q] == -1)
        else:
            # the sums are double; every weight of the path (T - 1 arcs, initial, final) was rounded to a float in log2
            # units once: half a unit of its size, and no weight here is larger than 16
            tol = 2.0 ** -24 * 16 * (T + 1)
            assert abs(score[q] - best.score[i]) <= tol
            assert abs(oracle.path_score(g, em[q], path[q, :T]) - best.score[i]) <= 2 * tol
            assert np.all(path[q, T:] == -1)
    for q in np.flatnonzero(lengths == 0):
        assert np.isneginf(za[q]) and np.isneginf(zb[q]) and np.isneginf(score[q]) and np.all(path[q] == -1)
    h.destroy()


@pytest.mark.parametrize("K,D,phones", [(3, 5, 1), (64, 7, 3), (65, 64, 12), (500, 65, 25), (1000, 300, 60)])
def test_objective_and_gradient_with_small_denominators(K, D, phones):
    """Both graphs' shares of a frame's gradient from one wave: few pdfs and many, sequences of one frame and of none."""
    import torch
    rng = np.random.default_rng(K)
    den = _graph(rng, K, 2, 0, D)
    num = wl.chain_graphs(rng, np.array([phones, 1, max(1, phones // 2), 1]), D)
    lengths = np.array([3 * phones + 2, 1, 3 * max(1, phones // 2), 0], dtype=np.int32)
    emis = (rng.standard_normal((4, int(lengths.max()) + 1, D)) * 2).astype(np.float32)
    hd, hn = fb.graph_from(den, D), fb.graph_from(num, D)
    fb.POISON_NEW_BUFFERS = True
    try:
        loss, zn, zd, grad = fb.lfmmi_loss_grad(hd, hn, torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda())
    finally:
        fb.POISON_NEW_BUFFERS = False
    torch.cuda.synchronize()
    zn, zd, grad = zn.cpu().numpy(), zd.cpu().numpy(), grad.cpu().numpy()
    live = np.flatnonzero(lengths > 0)
    ref = oracle.lfmmi(den, num, emis, lengths, sel=live)
    for got, want in ((zn[live], ref.logz_num), (zd[live], ref.logz_den)):
        both = np.isneginf(got) & np.isneginf(want)
        assert np.all(both | (np.abs(got - want) <= 1e-4 * np.maximum(1.0, np.abs(want))))
    assert np.abs(grad[live] - ref.grad).max() <= 1e-5
    assert np.all(grad[3] == 0) and np.isneginf(zn[3]) and np.isneginf(zd[3])
    hd.destroy(); hn.destroy()


@pytest.mark.parametrize("K,D", [(3, 2), (40, 9), (300, 20), (1000, 40)])
def test_nan_emissions_show(K, D):
    """NaN is not a legal emission, but a diverged network's must not come back as a finite loss and gradient: it is in
    both log Z, the state posteriors, the loss and the gradient of its sequence, and nowhere else."""
    import torch
    rng = np.random.default_rng(K)
    den = _graph(rng, K, 2, 0, D)
    den.init[:] = 0.0                                        # (every state is alive at every frame)
    num = wl.chain_graphs(rng, np.array([2, 3, 2]), D)
    lengths = np.array([20, 21, 19], dtype=np.int32)
    emis = (rng.standard_normal((3, 21, D)) * 2).astype(np.float32)
    hd, hn = fb.graph_from(den, D), fb.graph_from(num, D)
    l = torch.from_numpy(lengths).cuda()
    for frame, pdf in ((0, int(den.pdf[0])), (7, int(den.pdf[0])), (20, int(den.pdf[0])), (9, slice(None))):
        e = emis.copy()
        e[1, frame, pdf] = np.nan
        e = torch.from_numpy(e).cuda()
        a, _, za = fb.fb_alpha(hd, e, l)
        b, _, zb = fb.fb_beta(hd, e, l)
        gam, _ = fb.fb_posteriors(hd, a, b, l, 3, 21)
        loss, zn, zd, grad = fb.lfmmi_loss_grad(hd, hn, e, l)
        torch.cuda.synchronize()
        for z in (za, zb, zd):
            assert np.array_equal(np.isnan(z.cpu().numpy()), [False, True, False])
        assert np.isnan(loss.cpu().numpy()).all()
        if not isinstance(pdf, slice):                      # (a frame without a finite sum has posteriors 0, as in the general kernel)
            assert np.isnan(gam.cpu().numpy()[1]).any() and np.isnan(grad.cpu().numpy()[1]).any()
        else:
            assert np.isnan(zn.cpu().numpy()[1])
        for i in (0, 2):
            assert np.isfinite(gam.cpu().numpy()[i]).all() and np.isfinite(grad.cpu().numpy()[i]).all()
    hd.destroy(); hn.destroy()


def _dense_ring(rng, K, arcs, D, weight=0.0):
    """Every state alive at every frame: `arcs` arcs out of and into every state, the self-loop among them; the end
    weights spread, the start weights all alike."""
    src = np.tile(np.arange(K), arcs)
    dst = (src + np.repeat(np.arange(arcs), K)) % K
    logw = (weight - rng.exponential(size=src.size)).astype(np.float32)
    return wl.Graph(K, src.astype(np.int32), dst.astype(np.int32), logw, rng.integers(0, D, K).astype(np.int32),
                    np.zeros(K, np.float32), (-rng.exponential(size=K)).astype(np.float32))


@pytest.mark.parametrize("K,arcs", [(9, 2), (16, 4), (100, 2), (100, 9), (200, 2), (230, 6), (400, 3), (701, 2), (701, 5), (1000, 3)])
def test_masked_frames(K, arcs):
    """A frame whose emissions are all some large mask: the same posteriors on either side of it as those of the two
    pieces by themselves (what joins the pieces is lost in a sum of that size in any arithmetic, but neither the frames
    before nor the ones behind may lose their resolution), at the edges of the kernel's groups of frames."""
    import torch
    rng = np.random.default_rng(K + arcs)
    D, T = 13, 53
    g = _dense_ring(rng, K, arcs, D)
    masked = np.array([0, 1, 4, 7, 8, 9, 15, 16, 17, 24, 26, 27, 33, 48, 49, 51, 52], dtype=np.int64)
    B = masked.size
    lengths = np.full(B, T, dtype=np.int32)
    emis = (rng.standard_normal((B, T, D)) * 2).astype(np.float32)
    rows = np.arange(B)
    h = fb.graph_from(g, D)
    l = torch.from_numpy(lengths).cuda()
    before, behind = wl.Graph(**{**g.__dict__, "final": np.zeros(K, np.float32)}), wl.Graph(**{**g.__dict__, "init": np.zeros(K, np.float32)})
    zero = emis.copy()
    zero[rows, masked] = 0
    pieces = []
    for b, n in enumerate(masked):
        a = oracle.forward_backward(before, np.ascontiguousarray(zero[b:b + 1, :n + 1]), np.array([n + 1], np.int32))
        c = oracle.forward_backward(behind, np.ascontiguousarray(zero[b:b + 1, n:]), np.array([T - n], np.int32))
        # the piece that the place where the two halves of a best path meet lies in
        first = n > (T - 1) // 2
        part = zero[b:b + 1, :n + 1] if first else zero[b:b + 1, n:]
        best = oracle.viterbi(before if first else behind, np.ascontiguousarray(part), np.array([part.shape[1]], np.int32))
        pieces.append((a, c, first, best.score[0]))
    for mask in (np.float32(-1e20), np.float32(-1e25), np.finfo(np.float32).min):
        e = emis.copy()
        e[rows, masked] = mask
        e = torch.from_numpy(e).cuda()
        alpha, _, z = fb.fb_alpha(h, e, l)
        beta, cb, zb = fb.fb_beta(h, e, l)
        gam, _ = fb.fb_posteriors(h, alpha, beta, l, B, T)
        score, path = fb.fb_viterbi(h, e, l)
        torch.cuda.synchronize()
        z, zb, gam, score, path = (t.cpu().numpy() for t in (z, zb, gam, score, path))
        assert np.all(np.abs(score / float(mask) - 1) <= 1e-6)
        for b, n in enumerate(masked):
            a, c, first, best = pieces[b]
            p = path[b, :n + 1] if first else path[b, n:]
            part = zero[b, :n + 1] if first else zero[b, n:]
            # the sums are double, every weight is rounded to a float in log2 units once (none is larger than 16)
            assert abs(oracle.path_score(before if first else behind, part, p) - best) <= 2.0 ** -24 * 16 * (T + 1)
            assert np.isfinite(oracle.path_score(g, zero[b], path[b]))
            if mask > -1e30:                                # (below that a value counts as zero-bar in the sums)
                assert abs(z[b] / float(mask) - 1) <= 1e-6 and abs(zb[b] / float(mask) - 1) <= 1e-6
                assert np.abs(gam[b, :n] - a.gamma[0][:n]).max(initial=0.0) <= 1e-5
                assert np.abs(gam[b, n:] - c.gamma[0]).max() <= 1e-5
            else:
                assert np.isneginf(z[b]) and np.isneginf(zb[b]) and np.all(gam[b] == 0)
    h.destroy()


@pytest.mark.parametrize("K,arcs", [(16, 4), (230, 6), (701, 2)])
def test_large_weights(K, arcs):
    """The same where the large numbers are weights: start and end weights all -1e20 (or the lowest float, best path only)
    are a shift and nothing else, but for the emissions of the two frames that they are added to."""
    import torch
    rng = np.random.default_rng(K)
    D, T, B = 13, 40, 3
    g = _dense_ring(rng, K, arcs, D)
    g.final[:] = 0
    lengths = np.array([T, 17, 2], dtype=np.int32)
    emis = (rng.standard_normal((B, T, D)) * 2).astype(np.float32)
    emis[:, 0] = 0
    emis[np.arange(B), lengths - 1] = 0
    ref = oracle.forward_backward(g, emis, lengths)
    best = oracle.viterbi(g, emis, lengths)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    for size in (np.float32(-1e20), np.float32(-2e38)):
        ends = np.full(K, size, np.float32)
        h = fb.graph_from(wl.Graph(**{**g.__dict__, "init": ends, "final": ends}), D)
        alpha, _, z = fb.fb_alpha(h, e, l)
        beta, _, zb = fb.fb_beta(h, e, l)
        gam, _ = fb.fb_posteriors(h, alpha, beta, l, B, T)
        score, path = fb.fb_viterbi(h, e, l)
        torch.cuda.synchronize()
        z, zb, gam, score, path = (t.cpu().numpy() for t in (z, zb, gam, score, path))
        for b in range(B):
            Tb = int(lengths[b])
            if size > -1e30:
                assert abs(z[b] / (2 * float(size)) - 1) <= 1e-6 and abs(zb[b] / (2 * float(size)) - 1) <= 1e-6
                assert np.abs(gam[b, :Tb] - ref.gamma[b]).max() <= 1e-5
            else:
                assert np.isneginf(z[b]) and np.isneginf(zb[b]) and np.all(gam[b] == 0)
            # (the two halves of a path meet in the middle: each is the best one from there, whatever the ends' size)
            assert abs(score[b] / (2 * float(size)) - 1) <= 1e-6
            assert np.all(path[b, :Tb] >= 0) and np.isfinite(oracle.path_score(g, emis[b], path[b, :Tb]))
            if size > -1e30:
                assert abs(oracle.path_score(g, emis[b], path[b, :Tb]) - best.score[b]) <= 2.0 ** -24 * 16 * (T + 1)
        h.destroy()


@pytest.mark.parametrize("D", [2400, 2600])
def test_posteriors_of_many_pdfs(D):
    """600 states and D pdfs lie on either side of the size where large batches go to the workgroup-wide kernel: a
    sequence's posteriors are those it has by itself (the wave-wide kernel's), and sum to 1."""
    import torch
    rng = np.random.default_rng(D)
    g = _dense_ring(rng, 600, 3, D)
    B, N = 40, 210
    lengths = rng.integers(1, N + 1, B).astype(np.int32)
    lengths[0] = N
    emis = torch.from_numpy((rng.standard_normal((B, N, D)) * 2).astype(np.float32)).cuda()
    l = torch.from_numpy(lengths).cuda()
    h = fb.graph_from(g, D)
    alpha, beta = fb.fb_alpha(h, emis, l)[0], fb.fb_beta(h, emis, l)[0]
    gam, rho = fb.fb_posteriors(h, alpha, beta, l, B, N)
    for b in (0, 7, 39):
        gam1, rho1 = fb.fb_posteriors(h, alpha[b:b + 1].contiguous(), beta[b:b + 1].contiguous(), l[b:b + 1].contiguous(), 1, N)
        # the same sums in another order: a few units of single precision of numbers below 1
        assert float((gam1[0] - gam[b]).abs().max()) <= 1e-6 and float((rho1[0] - rho[b]).abs().max()) <= 1e-6
        real = rho[b, :lengths[b]].sum(dim=1).cpu().numpy()
        assert np.abs(real - 1).max() <= 1e-5 and float(rho[b, lengths[b]:].abs().sum()) == 0
    h.destroy()
