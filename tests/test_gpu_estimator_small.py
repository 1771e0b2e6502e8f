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
