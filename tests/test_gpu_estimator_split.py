"""The float estimator over its splits: threads of a workgroup, chunks of chains, groups that share a row's or a
bit's chains, and the three orders of the residual sums.

A launch of more than 256 instances takes the shape's own workgroup (256, 512 or 1024 threads), a smaller one
1024 threads: the results have to be the same bit for bit.  Against the oracle's estimates on the same final
states the tolerance follows from the float32 energies: with u = 2^-24, a residual of 2 nt + 4 rounded terms is
off by about 4 sqrt(2 nt + 4) u (|y'| + 2 s sum |h| k) (four standard deviations), which moves f by
2 sum |r| dr / sigma^2, and an error d in the exponents moves a probability by at most d / 2.
"""
import numpy as np
import pytest

import workloads as W
from oracle import dmala as odm
from tests.helpers import gpu_available, run_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

OUTS = ("symbols", "marginals", "llrs", "best_energy", "final_state", "marginals_mc")


def _tolerance(prob, ks):
    s, Q, nt = prob.s, prob.Q, prob.Nt
    off = s * (Q - 1)
    A = np.abs(prob.H)
    rows = np.abs(prob.y) + off * A.sum(axis=1)
    tol = 0.0
    for k in ks:
        x = 2 * s * k - off
        r = np.abs(prob.y - prob.H @ x)
        dr = 4 * np.sqrt(2 * nt + 4) * 2.0 ** -24 * (rows + 2 * s * (A @ k))
        f = (r ** 2).sum() / prob.sigma2
        tol = max(tol, 2 * (r * dr).sum() / prob.sigma2 + 8 * len(r) ** 0.5 * 2.0 ** -24 * f)
    return tol / 2 + 1e-5


# one row; groups of 8, 4, 2 and 1; chunks of ragged chain counts; every residual order; H beside LDS; two rows per thread
@pytest.mark.parametrize("nt,nr,M,C,mode", [(1, 1, 4, 16, "is"), (3, 5, 16, 7, "is"), (8, 8, 64, 64, "list"), (9, 12, 16, 130, "is"),
                                            (16, 17, 64, 33, "mc"), (17, 17, 256, 48, "is"), (32, 32, 64, 100, "is"),
                                            (33, 40, 64, 37, "list"), (64, 64, 64, 50, "is"), (65, 66, 256, 20, "is"),
                                            (100, 127, 64, 50, "is"), (128, 128, 256, 16, "mc"), (4, 1100, 16, 20, "is")])
def test_estimates_do_not_depend_on_the_launch(nt, nr, M, C, mode):
    n = 257
    kw = dict(n_chains=C, n_iters=6, seed=11, trace=False, outputs=OUTS, llr_mode=mode)
    big = W.make_batch(nt, nr, M, 14.0, n, seed=nt)
    _, a = run_gpu(big, **kw)
    few = W.make_batch(nt, nr, M, 14.0, n, seed=nt)
    few.H, few.y, few.sigma2 = few.H[:2], few.y[:2], few.sigma2[:2]
    b32, b = run_gpu(few, **kw)
    for k in OUTS:
        np.testing.assert_array_equal(a[k][:2].view(np.uint8), b[k].view(np.uint8), err_msg=k)
    ants = sorted({0, nt // 2, nt - 1})
    prob = odm.Problem(b32.H[1], b32.y[1], b32.sigma2[1], M)
    ks = b["final_state"][1].reshape(C, 2 * nt).astype(np.int64)
    ref = odm.marginals_is(prob, ks, antennas=ants)
    tol = _tolerance(prob, ks)
    np.testing.assert_allclose(b["marginals"][1].reshape(nt, M)[ants], ref[ants], atol=tol)
    np.testing.assert_allclose(b["marginals_mc"][1].reshape(nt, M), odm.marginals_mc(prob.Q, nt, ks), atol=1e-6)


def test_flagged_instance_beside_a_sound_one():
    batch = W.make_batch(6, 6, 64, 14.0, 2, seed=3)
    batch.H[0, 1, 2] = np.inf
    _, a = run_gpu(batch, 24, 6, 2, trace=False, outputs=OUTS)
    assert (a["symbols"][0] == -1).all() and (a["symbols"][1] >= 0).all()
    for k in ("marginals", "llrs", "marginals_mc"):
        assert np.isnan(a[k][0]).all() and np.isfinite(a[k][1]).all(), k
