"""What this library's users have it do: the calls, sizes and inputs that its speed is judged by.

The paths are the public ones of ``paper_2112_00709_amd``:

``fb``       fb_alpha, fb_beta and fb_posteriors, the forward-backward of a batch
``lfmmi``    lfmmi_loss_grad with the workspace and the gradient buffer kept by the caller
``train``    a training step on new utterances: their numerator graphs are built (every minibatch has its own),
             the objective is taken through autograd and the gradient of the network's output comes back
``viterbi``  fb_viterbi: forced alignment on small graphs, best path on a large one
``leaky``    fb_leaky_posteriors, the comparison mode

Graphs: ``random`` (a shared graph, out-degree 1 + Poisson, destinations uniform, or with ``zipf`` skewed by a
Zipf(1.1) law, so that a few hub states have thousands of arcs), ``chain`` (one left-to-right chain of three states a
phone per utterance) and ``ctc`` (one connectionist-temporal-classification topology per utterance).  Emissions are
normal pseudo-log-likelihoods with the standard deviation ``sigma`` (for ``ctc``: log-softmax of such scores).
"""
import math

import numpy as np
import torch

import paper_2112_00709_amd as fb
from paper_2112_00709_amd import autograd as fb_autograd

NEG_INF = np.float32(-np.inf)


def listed():
    return [
        # one short utterance on a graph of a few states: nothing but latency and launches (an interactive call, a unit test)
        dict(name="fb_tiny", path="fb", graph="random", K=16, degree=3.0, zipf=False, B=1, Nmin=50, Nmax=50, D=16, sigma=1.0,
             state=True),
        # posteriors of a minibatch of short utterances on their own alignment graphs
        dict(name="fb_chains", path="fb", graph="chain", Lmin=10, Lmax=40, stretch=1.2, B=32, D=84, sigma=2.0, state=True),
        # a phone-loop sized shared graph, odd sizes, state posteriors wanted as well
        dict(name="fb_state", path="fb", graph="random", K=701, degree=5.0, zipf=False, B=23, Nmin=61, Nmax=211, D=97,
             sigma=2.0, state=True),
        # a denominator graph over training chunks of 1.5 seconds, all of one length
        dict(name="fb_mid", path="fb", graph="random", K=2000, degree=10.0, zipf=False, B=64, Nmin=150, Nmax=150, D=84,
             sigma=2.0, state=False),
        # the largest denominator graph, hub states and thousands of outputs, utterances of unequal length
        dict(name="fb_large", path="fb", graph="random", K=6000, degree=10.0, zipf=True, B=128, Nmin=100, Nmax=500, D=3000,
             sigma=3.0, state=False),
        # objective and gradient of a handful of short utterances with a small denominator
        dict(name="lfmmi_small", path="lfmmi", K=307, degree=4.0, zipf=False, B=8, Lmin=5, Lmax=20, stretch=1.2, D=40,
             sigma=2.0, host_lengths=False),
        # objective and gradient of a large batch of equally long utterances; sizes of the paper's own benchmark
        dict(name="lfmmi_equal", path="lfmmi", K=3022, degree=16.87, zipf=False, B=128, Lmin=151, Lmax=151, N=700, D=84,
             sigma=2.0, host_lengths=True),
        # objective and gradient of a large batch of utterances of unequal length, thousands of outputs
        dict(name="lfmmi_large", path="lfmmi", K=6000, degree=10.0, zipf=True, B=128, Lmin=30, Lmax=150, stretch=1.2, D=3000,
             sigma=3.0, host_lengths=False),
        # a training step: numerators of this minibatch built, objective, gradient
        dict(name="train_step", path="train", K=3022, degree=16.87, zipf=False, B=64, Lmin=15, Lmax=45, stretch=1.2, D=84,
             sigma=2.0, host_lengths=True),
        # forced alignment of label sequences of unequal length
        dict(name="viterbi_align", path="viterbi", graph="ctc", Lmin=10, Lmax=80, stretch=1.3, B=32, D=129, sigma=2.0),
        # best path through a large graph
        dict(name="viterbi_den", path="viterbi", graph="random", K=6000, degree=10.0, zipf=True, B=128, Nmin=100, Nmax=500,
             D=3000, sigma=3.0),
        # the approximate denominator on a batch the size of the paper's benchmark
        dict(name="leaky_den", path="leaky", graph="random", K=3022, degree=16.87, zipf=False, B=128, Nmin=700, Nmax=700,
             D=84, sigma=2.0, leak=1e-5),
    ]


# --------------------------------------------------------------------------- more cases of the same ranges

def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _shared(rng, K_lo, K_hi):
    K = _log_int(rng, K_lo, K_hi)
    degree = round(rng.uniform(3.0, min(17.0, 60000.0 / K)), 2)
    return dict(K=K, degree=degree, zipf=K >= 1500 and rng.random() < 0.5, sigma=round(rng.uniform(1.0, 3.0), 2))


def _frames(rng, lo, hi):
    Nmax = _log_int(rng, lo, hi)
    return dict(Nmin=Nmax if rng.random() < 0.3 else max(1, Nmax // rng.randint(2, 5)), Nmax=Nmax)


def draw(rng):
    path = rng.choice(["fb", "fb", "fb", "lfmmi", "lfmmi", "train", "viterbi", "viterbi", "leaky"])
    if path == "lfmmi" or path == "train":
        large = rng.random() < 0.6
        c = dict(path=path, **(_shared(rng, 1024, 6000) if large else _shared(rng, 100, 1000)))
        Lmax = _log_int(rng, 15, 150) if path == "lfmmi" else _log_int(rng, 15, 60)
        c.update(B=_log_int(rng, 4, 128 if path == "lfmmi" else 64), Lmin=Lmax if rng.random() < 0.3 else max(3, Lmax // rng.randint(2, 5)),
                 Lmax=Lmax, stretch=round(rng.uniform(1.05, 1.5 if Lmax < 100 else 1.2), 2), D=_log_int(rng, 40, 3000),
                 host_lengths=rng.random() < 0.5)
        return c
    if path in ("fb", "viterbi") and rng.random() < 0.35:
        Lmax = _log_int(rng, 12, 100)
        return dict(path=path, graph=rng.choice(["chain", "ctc"]), Lmin=max(3, Lmax // rng.randint(1, 5)), Lmax=Lmax,
                    stretch=round(rng.uniform(1.1, 1.5), 2), B=_log_int(rng, 1, 128), D=_log_int(rng, 40, 1000),
                    sigma=round(rng.uniform(1.0, 3.0), 2), **(dict(state=rng.random() < 0.5) if path == "fb" else {}))
    small = path == "fb" and rng.random() < 0.5
    c = dict(path=path, graph="random", **(_shared(rng, 12, 1000) if small else _shared(rng, 1024, 6000 if path != "leaky" else 4000)))
    c.update(B=_log_int(rng, 1, 32) if small else _log_int(rng, 16, 128), D=_log_int(rng, 16, 300) if small else _log_int(rng, 40, 3000),
             **_frames(rng, 30, 300 if small else 500))
    if path == "fb":
        c["state"] = small and rng.random() < 0.7
    if path == "leaky":
        c["leak"] = 1e-5
    return c


# --------------------------------------------------------------------------- graphs

def _random_graph(rng, K, degree, zipf, D):
    deg = 1 + rng.poisson(degree - 1.0, size=K)
    E = int(deg.sum())
    src = np.repeat(np.arange(K, dtype=np.int32), deg)
    if zipf:
        pmf = np.arange(1, K + 1, dtype=np.float64) ** -1.1
        dst = rng.permutation(K)[rng.choice(K, size=E, p=pmf / pmf.sum())]
    else:
        dst = rng.integers(0, K, size=E)
    e = rng.exponential(size=E)                      # log Dirichlet(1, ..., 1) per source
    logw = np.log(e / np.repeat(np.add.reduceat(e, np.cumsum(deg) - deg), deg))
    return dict(K=K, src=src, dst=dst.astype(np.int32), logw=logw.astype(np.float32),
                pdf=rng.integers(0, D, size=K).astype(np.int32), init=np.full(K, -np.log(K), np.float32),
                final=np.zeros(K, np.float32), state_off=None)


def _chain_graphs(rng, phones, D):
    off = np.concatenate([[0], np.cumsum(3 * phones)]).astype(np.int32)
    K, half = int(off[-1]), np.float32(math.log(0.5))
    s = np.arange(K, dtype=np.int32)
    src, dst = np.repeat(s, 2), np.stack([s, s + 1], axis=1).reshape(-1)
    keep = np.ones(2 * K, dtype=bool)
    keep[2 * (off[1:] - 1) + 1] = False              # the last state of a chain has its self-loop only
    init, final = np.full(K, NEG_INF), np.full(K, NEG_INF)
    init[off[:-1]] = 0.0
    final[off[1:] - 1] = half
    return dict(K=K, src=src[keep], dst=dst[keep], logw=np.full(int(keep.sum()), half, np.float32),
                pdf=rng.integers(0, D, size=K).astype(np.int32), init=init, final=final, state_off=off)


def _ctc_graphs(rng, labels, D):
    off = np.concatenate([[0], np.cumsum(2 * labels + 1)]).astype(np.int32)
    K = int(off[-1])
    src, dst, pdf = [], [], np.zeros(K, np.int32)
    init, final = np.full(K, NEG_INF), np.full(K, NEG_INF)
    for b, L in enumerate(labels):
        k0, k1 = int(off[b]), int(off[b + 1])
        lab = rng.integers(1, D, size=int(L)).astype(np.int32)
        pdf[k0 + 1:k1:2] = lab
        s = np.arange(k0, k1, dtype=np.int32)
        skip = k0 + 1 + 2 * np.flatnonzero(lab[1:] != lab[:-1]).astype(np.int32)
        src += [s, s[:-1], skip]
        dst += [s, s[1:], skip + 2]
        init[k0:k0 + 2] = 0.0
        final[k1 - 2:k1] = 0.0
    src, dst = np.concatenate(src), np.concatenate(dst)
    return dict(K=K, src=src.astype(np.int32), dst=dst.astype(np.int32), logw=np.zeros(src.size, np.float32), pdf=pdf,
                init=init, final=final, state_off=off)


def _spread(case, lo, hi):
    """B whole numbers evenly over [lo, hi], the largest among them: every seed's batch has the same sizes in it."""
    return np.rint(np.linspace(hi, lo, case["B"])).astype(np.int64)


def _utterances(rng, case):
    """Chain or label-sequence graphs of a batch and the lengths that go with them."""
    L = rng.permutation(_spread(case, case["Lmin"], case["Lmax"]))
    ctc = case.get("graph") == "ctc"
    g = _ctc_graphs(rng, L, case["D"]) if ctc else _chain_graphs(rng, L, case["D"])
    states = np.diff(g["state_off"])
    lengths = np.full(case["B"], case["N"]) if "N" in case else np.rint(case["stretch"] * states)
    return g, lengths.astype(np.int32)


def _draw_inputs(case, seed):
    """(shared graph or None, packed graphs or None, lengths), host side, from the seed alone."""
    rng = np.random.default_rng(seed)
    shared = packed = lengths = None
    if "K" in case:
        shared = _random_graph(rng, case["K"], case["degree"], case["zipf"], case["D"])
    if "Lmax" in case:
        packed, lengths = _utterances(rng, case)
    else:
        lengths = rng.permutation(_spread(case, case["Nmin"], case["Nmax"])).astype(np.int32)
    return shared, packed, lengths


def _create(g, D):
    return fb.fb_graph_create(g["K"], g["src"], g["dst"], g["logw"], g["pdf"], g["init"], g["final"], D, g["state_off"])


def prepare(case, seed):
    shared, packed, lengths = _draw_inputs(case, seed)
    st = dict(case=case, lengths_host=lengths)
    B, N, D = case["B"], int(lengths.max()), case["D"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    emis = torch.randn((B, N, D), generator=gen, device="cuda", dtype=torch.float32).mul_(case["sigma"])
    if case.get("graph") == "ctc":
        emis = torch.log_softmax(emis, dim=2)
    st["emis"], st["lengths"] = emis, torch.from_numpy(lengths).cuda()
    if case["path"] in ("lfmmi", "train"):
        st["den"] = _create(shared, D)
        if case["path"] == "train":
            st["numerators"] = packed                # what the data loader hands over with the utterances
            st["emis"] = emis.requires_grad_(True)
        else:
            st["num"] = _create(packed, D)
            st["ws"] = torch.empty(fb.fb_lfmmi_workspace_bytes(st["den"], st["num"], B, N, D), dtype=torch.uint8, device="cuda")
            st["grad"] = torch.empty((B, N, D), dtype=torch.float32, device="cuda")
    else:
        st["g"] = _create(packed if packed is not None else shared, D)
        if case["path"] == "viterbi":
            need = fb.lib().fb_viterbi_workspace_bytes(st["g"].handle, B, N)
            st["ws"] = torch.empty(int(need), dtype=torch.uint8, device="cuda")
        elif case["path"] == "leaky":
            st["ws"] = torch.empty(fb.fb_leaky_workspace_bytes(st["g"], B, N), dtype=torch.uint8, device="cuda")
    return st


# --------------------------------------------------------------------------- one pass

def run(st):
    case, emis, lengths = st["case"], st["emis"], st["lengths"]
    path = case["path"]
    if path == "fb":
        alpha, _, logz = fb.fb_alpha(st["g"], emis, lengths)
        beta, _, logz_back = fb.fb_beta(st["g"], emis, lengths)
        B, N, _ = emis.shape
        state_post, pdf_post = fb.fb_posteriors(st["g"], alpha, beta, lengths, B, N, want_state=case["state"])
        # (alpha and beta rows are given up to a shift of each row, which is the library's choice: what does not depend
        # on it is compared)
        out = {"logz": logz, "logz_back": logz_back, "pdf_post": pdf_post}
        if case["state"]:
            out["state_post"] = state_post
        return out
    if path == "lfmmi":
        loss, zn, zd, grad = fb.lfmmi_loss_grad(st["den"], st["num"], emis, lengths, ws=st["ws"], grad=st["grad"],
                                                lengths_host=st["lengths_host"] if case["host_lengths"] else None)
        return {"loss": loss, "logz_num": zn, "logz_den": zd, "grad": grad}
    if path == "train":
        emis.grad = None
        num = _create(st["numerators"], case["D"])
        loss, zn, zd = fb_autograd.lfmmi_loss(emis, lengths, st["den"], num,
                                              lengths_host=st["lengths_host"] if case["host_lengths"] else None)
        loss.backward()
        torch.cuda.current_stream().synchronize()    # a graph may go only when nothing uses it any more
        num.destroy()
        return {"loss": loss.detach(), "logz_num": zn, "logz_den": zd, "grad": emis.grad}
    if path == "viterbi":
        score, best = fb.fb_viterbi(st["g"], emis, lengths, ws=st["ws"])
        return {"score": score, "path": best}
    logz, post = fb.fb_leaky_posteriors(st["g"], emis, lengths, case["leak"], ws=st["ws"])
    return {"logz": logz, "pdf_post": post}


# --------------------------------------------------------------------------- what a pass cannot do without

def _sizes(case):
    """(frames of the batch, frames of the longest, states x frames and arcs x frames of the packed graphs)."""
    if "Lmax" not in case:
        return float(_spread(case, case["Nmin"], case["Nmax"]).sum()), case["Nmax"], 0.0, 0.0
    L = _spread(case, case["Lmin"], case["Lmax"])
    ctc = case.get("graph") == "ctc"
    states = 2 * L + 1 if ctc else 3 * L
    frames = np.full(case["B"], case["N"]) if "N" in case else np.rint(case["stretch"] * states)
    kf = float((states * frames).sum())
    return float(frames.sum()), int(frames.max()), kf, (2.5 if ctc else 2.0) * kf


def work(case):
    frames, longest, pk, pa = _sizes(case)
    B, D, path = case["B"], case["D"], case["path"]
    K, E = case.get("K", 0), case.get("K", 0) * case.get("degree", 0.0)
    used = K * (1.0 - (1.0 - 1.0 / D) ** K) * D / max(K, 1) if K else 0.0     # pdfs that some state of the shared graph is tied to
    emis = 4.0 * frames * used if K else 4.0 * pk
    if path in ("lfmmi", "train"):
        # emissions read, gradient written (rows of padding too), vectors of neither graph needed in memory
        return {"bytes": emis + 4.0 * pk + 4.0 * B * longest * D + 12.0 * E, "flops": 4.0 * (frames * E + pa)}
    kf = frames * K if K else pk
    arcs = frames * E if K else pa
    if path == "viterbi":
        return {"bytes": emis + 4.0 * B * longest + 12.0 * E, "flops": 2.0 * arcs}
    if path == "leaky":
        return {"bytes": emis + 4.0 * B * longest * D + 12.0 * E, "flops": 4.0 * arcs}
    # alpha and beta are results of two calls and inputs of a third; every call reads the emissions it needs
    states = 4.0 * kf if case["state"] else 0.0
    return {"bytes": 2.0 * emis + 16.0 * kf + 4.0 * B * longest * D + states + 12.0 * E, "flops": 4.0 * arcs}


def tolerance(case):
    """About four times the largest difference seen between these paths and the same sums in 64 bits, over the listed
    cases and some forty drawn ones."""
    path = case["path"]
    if path == "viterbi":
        # seen: scores 1e-16 with double vectors (small graphs), 5e-8 with float vectors, the same path every time; paths
        # within rounding of the best one are as good
        return {"rel": 2e-7, "max": 3e-7, "differ": 2e-3} if "K" in case else {"rel": 1e-12, "max": 1e-12, "differ": 1e-3}
    if path in ("lfmmi", "train"):
        return {"rel": 8e-7, "max": 2e-5}            # seen: 1.9e-7, 4.6e-6
    if path == "leaky":
        return {"rel": 1e-6, "max": 1e-5}            # seen: 1.5e-7, 1e-6 (a smaller sample), two sides compared
    if "K" in case:
        return {"rel": 2.7e-6, "max": 2.5e-5}        # seen: 6.7e-7, 5.7e-6
    return {"rel": 3.5e-6, "max": 5e-5}              # rows of long chains leave as floats; seen: 8.1e-7, 1.3e-5
