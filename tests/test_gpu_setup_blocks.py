"""The blocked Gauss-Jordan setup: every workgroup size, blocks of 16 and their remainders, alone and in a plan.

A large launch takes smaller workgroups than a small one; the packed matrices follow from float64 values that differ
by rounding at most, so the chains have to be the same; against the oracle's they may part at near-ties only.
"""
import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_available, run_gpu, run_oracle, compare_chains, EPS32, eps32_mh

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

OUTS = ("symbols", "final_state", "accept_count")


def _head(batch, n):
    batch.H, batch.y, batch.sigma2 = batch.H[:n], batch.y[:n], batch.sigma2[:n]
    return batch


@pytest.mark.parametrize("nt,nr,n", [(1, 1, 1025), (4, 3, 1025), (15, 17, 1030), (16, 16, 1025), (17, 33, 1026), (31, 40, 1025),
                                     (32, 32, 1030), (33, 33, 514), (47, 60, 513), (48, 48, 513), (49, 65, 515), (64, 64, 513)])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_large_launches_equal_small_ones(nt, nr, n, precision):
    kw = dict(n_chains=16, n_iters=8, seed=7, precision=precision, trace=False, outputs=OUTS)
    _, a = run_gpu(W.make_batch(nt, nr, 16, 16.0, n, seed=nt), **kw)
    _, b = run_gpu(_head(W.make_batch(nt, nr, 16, 16.0, n, seed=nt), 4), **kw)
    for k in OUTS:
        np.testing.assert_array_equal(a[k][:4], b[k], err_msg=k)


@pytest.mark.parametrize("nt,nr", [(1, 2), (15, 15), (16, 18), (17, 17), (33, 33), (63, 64), (65, 70), (80, 80), (112, 113), (127, 128)])
def test_chains_follow_the_oracle(nt, nr):
    C, T = 4, 10
    b, g = run_gpu(W.make_batch(nt, nr, 16, 16.0, 2, seed=nt), C, T, 5)
    for i in range(2):
        o = run_oracle(b, i, C, T, 5, estimators=False)
        _, _, bad = compare_chains(g["trace_hash"][i], o, EPS32[0], eps32_mh)
        assert not bad


def test_plan_equals_single_calls():
    import torch
    import paper_2407_06042_amd as dm
    c3 = W.c3_uneven(600)
    H, y, s2 = dm.pack_uneven(c3["H"], c3["y"], c3["sigma2"])
    plan = dm.Plan(c3["shapes"], 16, 8, 5, outputs=("final_state",))
    o = plan(H, y, s2)
    torch.cuda.synchronize()
    fs = o["final_state"].cpu().numpy()
    seen, at = {}, 0
    for i, (nt, nr, M) in enumerate(c3["shapes"]):
        n = 16 * 2 * nt
        if seen.get((nt, nr), 0) < 2:
            seen[(nt, nr)] = seen.get((nt, nr), 0) + 1
            Hi, yi, si = dm.device_inputs(c3["H"][i][None], c3["y"][i][None], np.array([c3["sigma2"][i]]))
            r = dm.Detector(1, nt, nr, M, 16, 8, 5, counter_base=i, outputs=("final_state",))(Hi, yi, si)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(fs[at:at + n], r["final_state"].cpu().numpy().reshape(-1), err_msg=str((i, nt, nr, M)))
        at += n
