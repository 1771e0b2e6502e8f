"""An instance's packed block (matrices, vectors, features) is the same bytes in any launch.

The setup's workgroup size follows from the number of instances and from plan or direct launch; its float64 sums and
their order must not.  float64 problems store the sums themselves, so that one rounding shows.
"""
import numpy as np
import pytest

import workloads as W
from tests.helpers import PREC_NP, gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

C, T = 4, 1


def _run(dm, d, H, y, s2):
    import torch
    d.ws.zero_()
    d(H, y, s2)
    torch.cuda.synchronize()
    at = (-d.ws.data_ptr()) % 256
    return d.ws[at:].cpu().numpy()


def _blocks(dm, b, nt, nr, M, precision, picks):
    """Per pick its block alone (one instance), the block's size, and the big launch's and the plan's blocks."""
    H, y, s2 = dm.device_inputs(b.H, b.y, b.sigma2, precision)
    n = len(b.sigma2)
    one = [_run(dm, dm.Detector(1, nt, nr, M, C, T, 1, precision), H[i:i + 1], y[i:i + 1], s2[i:i + 1]) for i in picks]
    big = _run(dm, dm.Detector(n, nt, nr, M, C, T, 1, precision), H, y, s2)
    plan = _run(dm, dm.Plan([(nt, nr, M)] * n, C, T, 1, precision), H.reshape(-1), y.reshape(-1), s2)
    # a block starts with |y|^2 (float64): the second instance's place is the block's size
    second = _run(dm, dm.Detector(1, nt, nr, M, C, T, 1, precision), H[1:2], y[1:2], s2[1:2])
    heads = big[:len(big) // 256 * 256].reshape(-1, 256)[:, :8]
    size = 256 * int(np.nonzero(np.all(heads == second[:8], axis=1))[0][0])
    return one, size, big, plan


@pytest.mark.parametrize("nt,nr,n,precision", [(1, 3, 1025, "fp64"), (5, 9, 1030, "fp64"), (16, 16, 1025, "fp64"),
                                               (17, 29, 1025, "fp64"), (32, 40, 1025, "fp64"), (8, 8, 1025, "fp32"),
                                               (32, 33, 1025, "bf16"), (48, 50, 513, "fp32"), (64, 64, 513, "fp16"),
                                               (65, 70, 6, "fp32"), (128, 128, 6, "bf16")])
def test_blocks_do_not_depend_on_the_launch(nt, nr, n, precision):
    import paper_2407_06042_amd as dm
    b = W.make_batch(nt, nr, 16, 16.0, n, seed=nt).as_precision(PREC_NP[precision])
    picks = [0, 2, n // 2, n - 1]
    one, size, big, plan = _blocks(dm, b, nt, nr, 16, precision, picks)
    assert size > 256
    for i, o in zip(picks, one):
        for name, ws in (("large", big), ("plan", plan)):
            np.testing.assert_array_equal(ws[i * size:(i + 1) * size], o[:size], err_msg="%s launch, instance %d" % (name, i))
