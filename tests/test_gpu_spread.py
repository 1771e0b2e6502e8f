"""Kernels chosen by the size of a launch or of its problems, against the ones they stand in for.

Up to 8 antennas the 32-dimension layout leaves its
padding tile out: no other kernel runs these sizes, so they are compared with the float64 oracle's chains.
"""
import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_available, run_gpu, run_oracle, compare_chains, EPS32, eps32_mh

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

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
