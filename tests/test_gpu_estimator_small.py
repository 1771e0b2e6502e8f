"""The estimator on few chains and small problems: the groups that share chains have one each at least, and a launch of
at most one workgroup per CU takes the larger workgroups only where they are the faster ones."""
import numpy as np
import pytest

import workloads as W
from oracle import dmala as odm
from tests.helpers import gpu_available, run_gpu
from tests.test_gpu_estimator_chunks import _time
from tests.test_gpu_estimator_split import OUTS, _tolerance

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("nt,nr,M,C,mode", [(1, 1, 4, 1, "is"), (3, 4, 16, 2, "is"), (2, 2, 256, 3, "is"), (8, 9, 64, 5, "list"),
                                            (33, 33, 16, 1, "mc"), (16, 16, 256, 9, "is"), (24, 24, 64, 32, "is"),
                                            (24, 25, 256, 128, "is")])
def test_few_chains(nt, nr, M, C, mode):
    kw = dict(n_chains=C, n_iters=4, seed=3, trace=False, outputs=OUTS, llr_mode=mode)
    big = W.make_batch(nt, nr, M, 14.0, 257, seed=nt)
    _, a = run_gpu(big, **kw)
    few = W.make_batch(nt, nr, M, 14.0, 257, seed=nt)
    few.H, few.y, few.sigma2 = few.H[:2], few.y[:2], few.sigma2[:2]
    b32, b = run_gpu(few, **kw)
    for k in OUTS:
        np.testing.assert_array_equal(a[k][:2].view(np.uint8), b[k].view(np.uint8), err_msg=k)
    prob = odm.Problem(b32.H[1], b32.y[1], b32.sigma2[1], M)
    ks = b["final_state"][1].reshape(C, 2 * nt).astype(np.int64)
    ants = sorted({0, nt - 1})
    np.testing.assert_allclose(b["marginals"][1].reshape(nt, M)[ants], odm.marginals_is(prob, ks, antennas=ants)[ants],
                               atol=_tolerance(prob, ks))


@pytest.mark.parametrize("nt,M,C", [(3, 256, 1), (8, 256, 16), (16, 256, 32), (8, 64, 16), (4, 4, 64)])
def test_a_launch_within_the_chip_is_not_slower(nt, M, C):
    """256 problems, one per CU, against 257 of them (with 1024 threads for all of them 1.1 to 1.7 times as long)."""
    a, b = min(_time(nt, nt, M, C, 256) for _ in range(3)), min(_time(nt, nt, M, C, 257) for _ in range(3))
    print("%.1f us, of 257 %.1f" % (1e3 * a, 1e3 * b), flush=True)
    assert a < 1.08 * b


@pytest.mark.parametrize("nt,nr,M,C,n", [(33, 33, 256, 40, 257), (64, 64, 256, 1024, 2), (65, 65, 256, 33, 257), (70, 71, 64, 20, 257),
                                         (20, 21, 256, 100, 2), (5, 5, 4, 700, 2)])
def test_histogram_counts(nt, nr, M, C, n):
    """The Monte Carlo marginals are the final states' counts, one or two rows a thread, up to the largest chain count."""
    _, a = run_gpu(W.make_batch(nt, nr, M, 14.0, n, seed=nt), n_chains=C, n_iters=2, seed=3, trace=False,
                   outputs=("final_state", "marginals_mc"))
    Q = int(round(M ** 0.5))
    for i in (0, n - 1):
        k = a["final_state"][i].reshape(C, nt, 2).astype(np.int64)
        ref = np.stack([np.bincount(k[:, m, 0] * Q + k[:, m, 1], minlength=M) for m in range(nt)]) / np.float32(C)
        np.testing.assert_array_equal(a["marginals_mc"][i].reshape(nt, M), ref.astype(np.float32))


def test_row_forms_side_by_side_in_a_plan():
    """256-QAM classes of one and of two rows per thread, and another alphabet, in one plan's launches."""
    import torch
    import paper_2407_06042_amd as dm
    shapes = [(64, 64, 256)] * 2 + [(65, 66, 256)] * 3 + [(40, 41, 256)] * 2 + [(128, 128, 256), (70, 70, 64), (5, 6, 256)]
    C, T, seed = 40, 3, 5
    bs = [W.make_batch(nt, nr, M, 20.0, 1, seed=i).as_precision(np.float32) for i, (nt, nr, M) in enumerate(shapes)]
    H, y, sig = dm.pack_uneven([b.H[0] for b in bs], [b.y[0] for b in bs], np.array([b.sigma2[0] for b in bs]))
    outs = ("symbols", "marginals", "llrs", "best_energy", "marginals_mc")
    res = {k: v.cpu().numpy() for k, v in dm.Plan(shapes, C, T, seed, outputs=outs)(H, y, sig).items()}
    at = dict.fromkeys(outs, 0)
    for i, (nt, nr, M) in enumerate(shapes):
        u = dm.Detector(1, nt, nr, M, C, T, seed, outputs=outs, counter_base=i)(*dm.device_inputs(bs[i].H, bs[i].y, bs[i].sigma2))
        torch.cuda.synchronize()
        for k in outs:
            v = u[k].cpu().numpy().reshape(-1)
            np.testing.assert_array_equal(v, res[k][at[k]:at[k] + v.size], err_msg="%s of problem %d" % (k, i))
            at[k] += v.size


def _time_of(nt, nr, M, C, n, outputs):
    """Median time of the estimator's kernel for n instances (no transitions)."""
    import torch
    import paper_2407_06042_amd as dm
    g = torch.Generator(device="cuda").manual_seed(1)
    H = torch.randn(n, nt, nr, dtype=torch.complex64, device="cuda", generator=g) / nr ** 0.5
    y = torch.randn(n, nr, dtype=torch.complex64, device="cuda", generator=g)
    d = dm.Detector(n, nt, nr, M, C, 0, 1, outputs=outputs)
    s2 = torch.full((n,), 0.1, device="cuda")
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in ev:
        e.record()
    ms = []
    for _ in range(12):
        d(H, y, s2, events=[e.cuda_event for e in ev])
        torch.cuda.synchronize()
        ms.append(ev[2].elapsed_time(ev[3]))
    return float(np.median(ms[2:]))


@pytest.mark.parametrize("nt,C,n", [(48, 32, 1000), (68, 32, 1000)])
def test_histogram_beside_the_sums(nt, C, n):
    """256-QAM with the Monte Carlo marginals: the counts are a few integer operations per chain beside the sums, and a
    store (kept beside the sums in registers they took 1.8 times the time of the sums alone with two rows per thread)."""
    a, b = (min(_time_of(nt, nt, 256, C, n, ("marginals", "best_energy") + mc) for _ in range(3)) for mc in ((), ("marginals_mc",)))
    print("%.1f us, with the histogram %.1f" % (1e3 * a, 1e3 * b), flush=True)
    assert b < 1.35 * a
