"""The sums behind a transition's log ratio have one order in every form of a kernel.

Seeds at which, with another order of a sum in one form, some chain decides a transition within rounding of a tie
the other way: spread launches against the layout's own kernel, and naive chains that propose their current state,
whose log ratio is exactly zero, at a uniform within 1e-6 of one.
"""
import numpy as np
import pytest

import workloads as W
from oracle import dmala as odm
from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("nt,M,snr,n,layout,T,seeds", [(16, 4, 6.0, 700, 1, 1500, (15, 56, 73)),
                                                       (32, 4, 6.0, 480, 10, 1000, (18, 477, 538)),
                                                       (16, 16, 14.0, 700, 1, 1500, (143, 204, 237)),
                                                       (64, 4, 6.0, 126, 8, 1000, (1, 2, 3))])
def test_spread_decides_ties_as_the_layout_kernel(nt, M, snr, n, layout, T, seeds):
    import torch
    import paper_2407_06042_amd as dm
    b = W.make_batch(nt, nt, M, snr, n, seed=nt).as_precision(np.float32)
    inputs = dm.device_inputs(b.H, b.y, b.sigma2)
    for seed in seeds:
        out = []
        for tc in (0, layout):
            o = dm.Detector(n, nt, nt, M, 32, T, seed, tile_config=tc, outputs=("final_state", "accept_count"))(*inputs)
            torch.cuda.synchronize()
            out.append({k: v.cpu().numpy() for k, v in o.items()})
        for k in out[0]:
            np.testing.assert_array_equal(out[0][k], out[1][k], err_msg="%s, seed %d" % (k, seed))


@pytest.mark.parametrize("nt,M,snr,seed,inst,chain", [(13, 256, 36.0, 2, 594, 54), (16, 64, 30.0, 3, 432, 52),
                                                      (16, 64, 30.0, 5, 208, 59), (25, 16, 24.0, 0, 307, 45)])
def test_a_proposal_of_the_current_state_is_accepted(nt, M, snr, seed, inst, chain):
    import torch
    import paper_2407_06042_amd as dm
    C, T = 64, 60
    b = W.make_batch(nt, nt, M, snr, 600, seed=nt).as_precision(np.float32)
    o = odm.detect(b.H[inst], b.y[inst], b.sigma2[inst], M, C, T, seed, instance=inst, variant="naive", trace=True,
                   estimators=False)["trace"]
    t = int(np.argmin(o["mh_margin"][:, chain]))
    assert o["log_ratio"][t, chain] == 0.0 and o["mh_margin"][t, chain] < 2e-6
    H, y, s2 = dm.device_inputs(b.H[inst:inst + 1], b.y[inst:inst + 1], b.sigma2[inst:inst + 1])
    got = dm.Detector(1, nt, nt, M, C, T, seed, "fp32", "naive", counter_base=inst, outputs=("accept_count",))(H, y, s2)
    torch.cuda.synchronize()
    assert got["accept_count"].cpu().numpy()[0, chain] == int(o["accept"][:, chain].sum())
