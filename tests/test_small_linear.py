"""Which small shared graphs run their sums on probabilities: the library's rule against its definition by strongly
connected components."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.csgraph as csg

import paper_2112_00709_amd as fb
import workloads as wl


def _expected(g):
    """Fewer than 4096 arcs, weights of ordinary size, rows of more than two arcs, one component with a cycle, everything within 24 steps of it."""
    log2 = np.concatenate([g.logw, g.init, g.final]).astype(np.float64) * 1.4426950408889634
    fin = log2[np.isfinite(log2)]
    if np.any(fin < -100) or np.any(fin > 40):
        return False
    rows = np.bincount(g.dst, minlength=g.K), np.bincount(g.src, minlength=g.K)
    if max(r.max() for r in rows) <= 2 or g.E >= 4096:
        return False
    live = np.isfinite(g.logw)
    A = sp.csr_matrix((np.ones(int(live.sum())), (g.src[live], g.dst[live])), shape=(g.K, g.K))
    n, label = csg.connected_components(A, directed=True, connection="strong")
    loops = A.diagonal() > 0
    size = np.bincount(label, minlength=n)
    cyclic = [c for c in range(n) if size[c] > 1 or loops[label == c].any()]
    if len(cyclic) != 1:
        return False
    # distances from the component's first state, as the library takes them
    root = int(np.flatnonzero(label == cyclic[0])[0])
    for M in (A, A.T.tocsr()):
        d = csg.shortest_path(M, unweighted=True, indices=root)
        if d[np.isfinite(d)].max() > 24:
            return False
    return True


def _graph(rng, K, deg, kind):
    n = max(1, int(K * deg))
    src, dst = rng.integers(0, K, n), rng.integers(0, K, n)
    logw = -rng.exponential(size=n)
    if kind == "ring":
        src, dst = np.concatenate([src, np.arange(K)]), np.concatenate([dst, (np.arange(K) + 1) % K])
    if kind == "sink":                                       # a state that keeps what it gets
        src, dst = np.concatenate([src[src != K - 1], [K - 1]]), np.concatenate([dst[src != K - 1], [K - 1]])
    if kind == "chain":                                      # left to right, with skips
        s = np.arange(K)
        src, dst = np.concatenate([s, s[:-1], s[:-2]]), np.concatenate([s, s[:-1] + 1, s[:-2] + 2])
    logw = -rng.exponential(size=src.size)
    if kind == "far":
        logw[0] = -75.0                                      # (108 binary orders)
    if kind == "dead":
        logw[rng.random(logw.size) < 0.3] = -np.inf
    return wl.Graph(K, src.astype(np.int32), dst.astype(np.int32), logw.astype(np.float32), rng.integers(0, 7, K).astype(np.int32),
                    np.zeros(K, np.float32), np.zeros(K, np.float32))


@pytest.mark.parametrize("kind", ["random", "ring", "sink", "chain", "far", "dead"])
def test_rule(kind):
    rng = np.random.default_rng(len(kind))
    seen = []
    for K, deg in [(3, 2), (5, 3), (16, 3), (17, 1.5), (40, 2), (64, 4), (90, 1.2), (150, 3), (300, 1.05), (300, 4), (700, 5), (1000, 3)] * 2:
        g = _graph(rng, K, deg, kind)
        h = fb.graph_from(g, 7, host_only=True)
        seen.append(bool(fb.fb_graph_small_linear(h)))
        assert seen[-1] == _expected(g), (kind, K, deg)
        h.destroy()
    assert any(seen) or kind in ("chain", "far", "sink")
    assert not all(seen) or kind == "ring"


def test_packed_and_large_graphs_are_not_taken():
    rng = np.random.default_rng(3)
    h = fb.graph_from(wl.chain_graphs(rng, np.array([3, 4]), 7), 7, host_only=True)
    assert fb.fb_graph_small_linear(h) == 0
    h.destroy()
    h = fb.graph_from(_graph(rng, 1100, 3, "random"), 7, host_only=True)
    assert fb.fb_graph_small_linear(h) == 0
    h.destroy()
