"""The leaky-HMM mode on large graphs (the recursion kernel of the exact path with the rank-one term, then the gradient
kernel) and where it hands sequences or graphs to the plain kernel."""
import numpy as np
import pytest

import workloads as wl
from oracle import leaky as oleaky

pytestmark = pytest.mark.gpu


def _compare(g, D, emis, lengths, leak):
    import torch

    import paper_2112_00709_amd as fb
    G = fb.graph_from(g, D)
    assert fb.fb_graph_linear_weights(G) == 2
    fb.POISON_NEW_BUFFERS = True
    try:
        logz, post = fb.fb_leaky_posteriors(G, torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda(), leak)
    finally:
        fb.POISON_NEW_BUFFERS = False
    torch.cuda.synchronize()
    logz, post = logz.cpu().numpy(), post.cpu().numpy()
    G.destroy()
    ref = oleaky.forward_backward(g, np.where(np.isnan(emis), np.float32(0), emis), lengths, leak)
    for b, T in enumerate(lengths):
        assert np.all(post[b, T:] == 0)
        if np.isneginf(ref.logz[b]):
            assert np.isneginf(logz[b]) and np.all(post[b] == 0)
            continue
        assert abs(logz[b] - ref.logz[b]) <= 1e-4 * max(1.0, abs(ref.logz[b]))
        assert np.abs(post[b] - ref.rho[b]).max() <= 1e-5


@pytest.mark.parametrize("leak", [0.0, 1e-5, 0.3, 1.0])
@pytest.mark.parametrize("K,D,kind", [(1025, 5, "uniform"), (1501, 84, "hubs"), (3500, 1000, "clones"), (1537, 84, "dense"), (3003, 90, "many")])
def test_large_graphs(K, D, kind, leak):
    """The kernel of up to 16 units a wave (the first two), the general one, and that of up to 20: rows over two lanes
    in both directions (dense), rows of one lane (many)."""
    rng = np.random.default_rng(K)
    deg = {"clones": 9.0, "dense": 19.0, "many": 9.6}.get(kind, 4.0)
    g = wl.random_graph(rng, K, D, mean_extra_deg=deg, zipf_s=1.1 if kind in ("hubs", "clones") else None)
    if kind == "clones":
        assert np.bincount(g.dst, minlength=K).max() > 2048       # a row of several clones
    g.init[:] = np.log(rng.dirichlet(np.full(K, 0.05))).astype(np.float32)    # most of the leak goes to a few states
    lengths = np.array([9, 1, 0, 2, 17], dtype=np.int32)
    emis = (rng.standard_normal((5, 18, D)) * 3).astype(np.float32)
    for b, T in enumerate(lengths):
        emis[b, T:] = np.nan
    _compare(g, D, emis, lengths, leak)


@pytest.mark.parametrize("K,D", [(6000, 2895), (6000, 2894), (5998, 2898)])
def test_the_largest_rows_that_fit_on_chip_memory(K, D):
    """Four vectors of K + 1 floats and three emission rows behind the first vector's 32 KB: 160 KB is what a workgroup
    has.  The fast form's workspace, larger than the plain kernel's, says that it serves the call."""
    import paper_2112_00709_amd as fb
    rng = np.random.default_rng(K + D)
    g = wl.random_graph(rng, K, D, mean_extra_deg=3.0)
    G = fb.graph_from(g, D)
    assert fb.fb_leaky_workspace_bytes(G, 2, 6) > (4 * 2 * 6 * K + 255) // 256 * 256
    G.destroy()
    emis = (rng.standard_normal((2, 6, D)) * 2).astype(np.float32)
    _compare(g, D, emis, np.array([6, 3], dtype=np.int32), 1e-3)


def test_sequences_that_leave_the_range():
    """An unused pdf far above the others: the fast form gives those sequences up, the plain kernel redoes them, the
    rest stay; a frame nobody can emit has no path."""
    rng = np.random.default_rng(3)
    g = wl.random_graph(rng, 1200, 40, mean_extra_deg=5.0)
    g.pdf[:] = g.pdf % 20
    emis = (rng.standard_normal((4, 12, 40)) * 2).astype(np.float32)
    emis[1, 3:5, 30] = 200.0
    emis[2, 6, :] = -np.inf
    _compare(g, 40, emis, np.array([12, 12, 12, 7], dtype=np.int32), 1e-3)


def test_states_without_arcs_out():
    """Going backward such a state gets the leak and nothing else: the plain kernel's."""
    rng = np.random.default_rng(4)
    g = wl.random_graph(rng, 1300, 30, mean_extra_deg=5.0)
    keep = (g.src % 50) != 7
    g = wl.Graph(g.K, g.src[keep], g.dst[keep], g.logw[keep], g.pdf, g.init, g.final)
    emis = (rng.standard_normal((3, 10, 30)) * 2).astype(np.float32)
    _compare(g, 30, emis, np.array([10, 4, 8], dtype=np.int32), 0.01)


def test_workspace_for_one_sweep_is_enough():
    """Room for the plain kernel's rows only: that kernel serves the call; one byte less is refused."""
    import torch

    import paper_2112_00709_amd as fb
    rng = np.random.default_rng(6)
    g = wl.random_graph(rng, 1301, 30, mean_extra_deg=5.0)
    lengths = np.array([10, 4, 0], dtype=np.int32)
    emis = (rng.standard_normal((3, 10, 30)) * 2).astype(np.float32)
    G = fb.graph_from(g, 30)
    assert fb.fb_graph_linear_weights(G) == 2
    one = (4 * 3 * 10 * 1301 + 255) // 256 * 256
    assert one < fb.fb_leaky_workspace_bytes(G, 3, 10)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    ws = torch.full((one + 4096,), 77, dtype=torch.uint8, device="cuda")
    logz, post = fb.fb_leaky_posteriors(G, e, l, 1e-3, ws=ws[:one])
    torch.cuda.synchronize()
    assert bool((ws[one:] == 77).all())
    ref = oleaky.forward_backward(g, emis, lengths, 1e-3)
    for b, T in enumerate(lengths[:2]):
        assert abs(float(logz[b]) - ref.logz[b]) <= 1e-4 * max(1.0, abs(ref.logz[b]))
        assert np.abs(post[b].cpu().numpy() - ref.rho[b]).max() <= 1e-5
    with pytest.raises(fb.FBError) as err:
        fb.fb_leaky_posteriors(G, e, l, 1e-3, ws=ws[:one - 1])
    assert err.value.code == fb.FB_EINVAL
    G.destroy()
