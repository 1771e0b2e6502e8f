"""Kernels chosen by the size of a launch or of its problems, against the ones they stand in for.

Small launches spread each 16-chain block over more waves; the results have to be those of the layout's
own kernel (an explicit tile_config) bit for bit.  Up to 8 antennas the 32-dimension layout leaves its
padding tile out: no other kernel runs these sizes, so they are compared with the float64 oracle's chains.
"""
import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_available, run_gpu, run_oracle, compare_chains, EPS32, eps32_mh

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

ALL = ("symbols", "marginals", "llrs", "best_energy", "final_state", "accept_count", "train_rows")


# antennas at the edges of the 32-, 64- and 128-dimension layouts; ragged chain counts; every level count
@pytest.mark.parametrize("nt,nr,M,C", [(9, 9, 4, 16), (16, 18, 16, 20), (12, 12, 256, 33), (17, 17, 64, 16), (32, 33, 64, 32),
                                       (25, 31, 4, 40), (31, 31, 256, 17), (33, 40, 16, 24), (64, 64, 64, 48), (50, 50, 4, 16),
                                       (63, 70, 256, 16)])
@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
def test_spread_equals_the_layout_kernel(nt, nr, M, C, precision):
    layout = 1 if nt <= 16 else (10 if nt <= 32 else 8)
    batch = W.make_batch(nt, nr, M, 18.0, 3, seed=nt)
    for kw in (dict(trace=True), dict(trace=False, alpha_mult=2.0)):   # the 3-level window, then every level (Q >= 8)
        _, a = run_gpu(batch, C, 45, 5, precision, outputs=ALL, **kw)
        _, b = run_gpu(batch, C, 45, 5, precision, outputs=ALL, tile_config=layout, **kw)
        for k in a:
            np.testing.assert_array_equal(a[k].view(np.uint8), b[k].view(np.uint8), err_msg=k)


def test_spread_skips_a_flagged_instance():
    batch = W.make_batch(20, 20, 16, 18.0, 3, seed=1)
    batch.H[1, 2, 3] = np.nan
    _, a = run_gpu(batch, 24, 33, 5, outputs=ALL + ("status",))
    _, b = run_gpu(batch, 24, 33, 5, outputs=ALL + ("status",), tile_config=10)
    assert list(a["status"]) == [0, -3, 0]
    for k in a:
        np.testing.assert_array_equal(a[k].view(np.uint8), b[k].view(np.uint8), err_msg=k)


def test_small_plan_equals_single_calls():
    """A plan small enough for the spread kernels: every instance as the layout kernel gives it."""
    import torch
    import paper_2407_06042_amd as dm
    c3 = W.c3_uneven(24)
    H, y, s2 = dm.pack_uneven(c3["H"], c3["y"], c3["sigma2"])
    o = dm.Plan(c3["shapes"], 32, 40, 5)(H, y, s2)
    torch.cuda.synchronize()
    sym, fs = o["symbols"].cpu().numpy(), o["final_state"].cpu().numpy()
    s0 = f0 = 0
    for i, (nt, nr, M) in enumerate(c3["shapes"]):
        Hi, yi, si = dm.device_inputs(c3["H"][i][None], c3["y"][i][None], np.array([c3["sigma2"][i]]))
        layout = {16: 1, 32: 10, 64: 8, 128: 9}[nt]
        r = dm.Detector(1, nt, nr, M, 32, 40, 5, counter_base=i, tile_config=layout, outputs=("symbols", "final_state"))(Hi, yi, si)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(sym[s0:s0 + nt], r["symbols"].cpu().numpy()[0])
        np.testing.assert_array_equal(fs[f0:f0 + 64 * nt], r["final_state"].cpu().numpy().reshape(-1))
        s0 += nt
        f0 += 64 * nt


@pytest.mark.parametrize("nt,nr,M", [(1, 1, 4), (2, 3, 64), (7, 8, 16), (8, 8, 64), (8, 10, 256)])
@pytest.mark.parametrize("proposal", ["precond", "naive"])
def test_up_to_eight_antennas(nt, nr, M, proposal):
    """Chains identical to the oracle's up to near-ties (the rule of the parity tests)."""
    batch = W.make_batch(nt, nr, M, 16.0, 3, seed=3)
    b, g = run_gpu(batch, 20, 60, 77, "fp32", proposal)
    same = 0
    for i in range(3):
        o = run_oracle(b, i, 20, 60, 77, proposal)
        n_id, _, bad = compare_chains(g["trace_hash"][i], o, EPS32[0], eps32_mh)
        assert not bad
        same += n_id
        if n_id == 20:
            np.testing.assert_array_equal(g["symbols"][i], o["symbols"])
            np.testing.assert_allclose(g["marginals"][i], o["marginals"], atol=2e-4)
    assert same >= 50
