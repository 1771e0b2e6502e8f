"""Chunks of chains in the estimator's 512-thread workgroups, at shapes whose larger chunk would leave one workgroup a CU."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_available, run_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

SHAPES = [(48, 48, 64, 64), (67, 67, 16, 64), (62, 93, 64, 48)]
OUTS = ("symbols", "marginals", "llrs", "best_energy")


@pytest.mark.parametrize("nt,nr,M,C", SHAPES)
def test_large_launches_equal_small_ones(nt, nr, M, C):
    n = 257
    kw = dict(n_chains=C, n_iters=3, seed=11, trace=False, outputs=OUTS)
    _, a = run_gpu(W.make_batch(nt, nr, M, 14.0, n, seed=nt), **kw)
    few = W.make_batch(nt, nr, M, 14.0, n, seed=nt)
    few.H, few.y, few.sigma2 = few.H[:2], few.y[:2], few.sigma2[:2]
    _, b = run_gpu(few, **kw)
    for k in OUTS:
        np.testing.assert_array_equal(a[k][:2].view(np.uint8), b[k].view(np.uint8), err_msg=k)


def _time(nt, nr, M, C, n=4096):
    """Median time of the estimator's kernel for n instances (no transitions)."""
    import torch
    import paper_2407_06042_amd as dm
    g = torch.Generator(device="cuda").manual_seed(1)
    H = torch.randn(n, nt, nr, dtype=torch.complex64, device="cuda", generator=g) / nr ** 0.5
    y = torch.randn(n, nr, dtype=torch.complex64, device="cuda", generator=g)
    s2 = torch.full((n,), 0.1, device="cuda")
    d = dm.Detector(n, nt, nr, M, C, 0, 1)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in ev:
        e.record()
    ms = []
    for _ in range(12):
        d(H, y, s2, events=[e.cuda_event for e in ev])
        torch.cuda.synchronize()
        ms.append(ev[2].elapsed_time(ev[3]))
    return float(np.median(ms[2:]))


@pytest.mark.parametrize("nt,nr,M,C", SHAPES)
def test_no_step_at_the_lds_limit(nt, nr, M, C):
    """Two antennas less, whose chunk fits a CU twice, do almost the same work (one workgroup a CU took 1.5 times as long)."""
    a, b = _time(nt, nr, M, C), _time(nt - 2, nr - 2, M, C)
    print("%.3f ms, two antennas less %.3f" % (a, b), flush=True)
    assert a < 1.25 * b
