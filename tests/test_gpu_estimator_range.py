"""The float estimator where f = -||y - H x||^2 / sigma^2 comes near the largest float32.

Chains of no transitions keep their random initial states, which the oracle shares, so that its float64 estimates are
the reference.  One antenna: the rows' and the bits' chains are shared by eight threads.
"""
import numpy as np
import pytest

from oracle import dmala as odm
from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

H1 = np.ones((1, 1, 1), np.complex128)
Y1 = np.full((1, 1), 1000.0 + 500.0j)
SEED, C = 3, 33
FMAX = float(np.finfo(np.float32).max)


def _energies(M):
    """Energies of the chains' (initial) states."""
    p = odm.Problem(H1[0], Y1[0], 1.0, M)
    k = odm.dmala_sample(p, SEED, 0, C, 0)["k"]
    return np.array([float(np.ravel(p.energy(p.x_of(k[c:c + 1])))[0]) for c in range(C)]), k


def _run(M, sigma2, mode):
    import torch
    import paper_2407_06042_amd as dm
    H, y, s2 = dm.device_inputs(H1, Y1, np.array([sigma2]))
    d = dm.Detector(1, 1, 1, M, C, 0, SEED, llr_mode=mode, outputs=("marginals", "llrs", "final_state"))
    out = {k: v.cpu().numpy()[0] for k, v in d(H, y, s2).items()}
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("M", [4, 16, 64, 256])
@pytest.mark.parametrize("mode", ["is", "list"])
def test_bits_at_large_f(M, mode):
    """LLRs within 16 roundings (2^-24) of |f|, list LLRs at their limits as the oracle's."""
    E, k = _energies(M)
    sigma2 = float(np.float32(E.max() / 3.1e38))
    got = _run(M, sigma2, mode)
    np.testing.assert_array_equal(got["final_state"], k)
    p = odm.Problem(H1[0], Y1[0], sigma2, M)
    want = (odm.llr_is if mode == "is" else odm.llr_list)(p, k)
    tol = 16 * 2.0 ** -24 * 3.1e38 if mode == "is" else 0.0
    np.testing.assert_allclose(got["llrs"], want.reshape(got["llrs"].shape), rtol=0, atol=tol)
