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


def _overflow_case(M):
    """A channel so large that the energies of some chains, not the first's, exceed float32; |f| itself stays below 40."""
    Q = int(round(M ** 0.5))
    y = np.full((1, 1), np.sqrt(3.0 / (2.0 * (M - 1))) * (Q - 1) * (1.0 + 0.9j))
    p = odm.Problem(H1[0], y[0], 1.0, M)
    for seed in range(100):
        k = odm.dmala_sample(p, seed, 0, C, 0)["k"]
        E = np.array([float(np.ravel(p.energy(p.x_of(k[c:c + 1])))[0]) for c in range(C)])
        up = E[E > E[0] * 1.001]
        if len(up) > C // 4 and np.any(E[1:8] > E[0] * 1.001):
            break
    h = np.sqrt(FMAX / (0.5 * (E[0] + up.min())))
    single = lambda v: v.astype(np.complex64).astype(np.complex128)  # noqa: E731
    return seed, k, E * h * h > FMAX, single(H1 * h), single(y * h), float(np.float32(h * h * E.max() / 40.0))


# (at M = 4 the squared column norm itself overflows with them)
@pytest.mark.parametrize("M", [16, 64, 256])
@pytest.mark.parametrize("mode", ["is", "list"])
def test_chains_of_infinite_energy(M, mode):
    """Chains whose energy overflows add nothing.

    With one antenna every chain gives the same normalised marginals, so that the others' are the oracle's; the LLRs
    are the oracle's over the other chains.  |f| < 40 in float32, a dozen roundings of 2^-24: within 1e-4."""
    import torch
    import paper_2407_06042_amd as dm
    seed, k, over, H, y, sigma2 = _overflow_case(M)
    assert not over[0] and over[1:8].any() and over.sum() > C // 4
    d = dm.Detector(1, 1, 1, M, C, 0, seed, llr_mode=mode, outputs=("marginals", "llrs", "final_state", "best_energy"))
    got = {n: v.cpu().numpy()[0] for n, v in d(*dm.device_inputs(H, y, np.array([sigma2]))).items()}
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got["final_state"], k)
    p = odm.Problem(H[0], y[0], sigma2, M)
    np.testing.assert_allclose(got["marginals"], odm.marginals_is(p, k).reshape(got["marginals"].shape), rtol=0, atol=1e-4)
    if mode == "is":
        np.testing.assert_allclose(got["llrs"], odm.llr_is(p, k[~over]).reshape(got["llrs"].shape), rtol=1e-4, atol=1e-4)
    else:
        np.testing.assert_allclose(got["llrs"], odm.llr_list(p, k[~over]).reshape(got["llrs"].shape), rtol=1e-4, atol=1e-4)
