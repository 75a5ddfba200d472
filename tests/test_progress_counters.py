"""Progress counters of the LF-MMI recursion launches: a range's gradient launch runs on other streams as soon as the
range's counter says that its rows are written, so a workgroup may count only when all its waves' stores have arrived."""
import os
import re
import subprocess

import numpy as np
import pytest

import workloads as wl
from paper_2112_00709_amd import build

PROBE = r"""
#include "fb_device.h"
namespace fb {
__global__ __launch_bounds__(128) void probe(const RecParams P, float *rows, const float *values)
{
    if (threadIdx.x >= 64) rows[(size_t)blockIdx.x * 64 + threadIdx.x - 64] = values[threadIdx.x];   // a wave that does not count
    count_done(P);
}
}  // namespace fb
"""


def test_every_wave_waits_for_its_stores_before_the_workgroup_counts(tmp_path):
    """The code made for a kernel whose rows are stored by another wave than the one that counts: behind the store, the
    wave's wait for it, then the barrier, then the write-back and the count."""
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.check_call([build.HIPCC] + flags + ["--cuda-device-only", "-S", "-I", build.CSRC, "-I",
                                                   os.path.join(build.HERE, "..", "include"), str(src), "-o", str(out)])
    code = [m.group(0) for m in re.finditer(r"\bglobal_store_dword\b|s_waitcnt [^\n]*vmcnt\(0\)|\bs_barrier\b|\bbuffer_wbl2\b|"
                                            r"\bglobal_atomic_add\b", out.read_text())]
    kinds = [c.split()[0] for c in code]
    store, barrier = kinds.index("global_store_dword"), kinds.index("s_barrier")
    assert store < barrier and "s_waitcnt" in kinds[store:barrier]
    assert barrier < kinds.index("buffer_wbl2") < kinds.index("global_atomic_add")


@pytest.mark.gpu
@pytest.mark.parametrize("K,degree", [(40, 3), (301, 4), (700, 3)])
def test_ranges_released_by_counters_with_small_denominators(K, degree):
    """A batch large enough for ranges, its denominator in the small-graph kernel, no host lengths: every frame's gradient
    against the oracle, the workspace and the gradient poisoned before each call."""
    import torch

    import oracle
    import paper_2112_00709_amd as fb
    rng = np.random.default_rng(K)
    D = 23
    den = wl.random_graph(rng, K, D, mean_extra_deg=degree - 1)
    phones = rng.integers(2, 14, 40)
    num = wl.chain_graphs(rng, phones, D)
    lengths = (3 * phones + rng.integers(1, 20, 40)).astype(np.int32)
    emis = (rng.standard_normal((40, int(lengths.max()), D)) * 2).astype(np.float32)
    ref = oracle.lfmmi(den, num, emis, lengths)
    hd, hn = fb.graph_from(den, D), fb.graph_from(num, D)
    e, l = torch.from_numpy(emis).cuda(), torch.from_numpy(lengths).cuda()
    for _ in range(3):
        fb.POISON_NEW_BUFFERS = True
        try:
            loss, zn, zd, grad = fb.lfmmi_loss_grad(hd, hn, e, l)
        finally:
            fb.POISON_NEW_BUFFERS = False
        torch.cuda.synchronize()
        assert np.abs(grad.cpu().numpy() - ref.grad).max() <= 1e-5
        assert np.all(np.abs(zd.cpu().numpy() - ref.logz_den) <= 1e-4 * np.maximum(1.0, np.abs(ref.logz_den)))
    hd.destroy(); hn.destroy()
