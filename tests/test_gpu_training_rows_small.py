"""Training rows of up to 8 antennas, whose layout leaves out its padding tile: the features of every antenna, and
nothing beyond the rows."""
import numpy as np
import pytest

import workloads as W
from oracle import dmala as odm
from oracle import learned as ol
from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("nt,nr,M", [(1, 1, 4), (2, 3, 16), (7, 8, 64), (8, 8, 256)])
def test_rows_of_every_antenna(nt, nr, M):
    import torch
    import paper_2407_06042_amd as dm
    n, C = 3, 20
    b = W.make_batch(nt, nr, M, 18.0, n, seed=nt).as_precision(np.float32)
    det = dm.Detector(n, nt, nr, M, C, 5, 7, outputs=("final_state", "train_rows"))
    # the rows at the head of a larger buffer
    size = det.out["train_rows"].numel()
    buf = torch.full((3 * size,), -77.0, device="cuda")
    det._outs.train_rows = buf.data_ptr()
    k = det(*dm.device_inputs(b.H, b.y, b.sigma2))["final_state"].cpu().numpy().astype(np.int64)
    torch.cuda.synchronize()
    assert bool((buf[size:] == -77.0).all())
    rows = buf[:size].cpu().numpy().reshape(n, C, nt, 12)
    for i in range(n):
        prob = odm.Problem(b.H[i], b.y[i], b.sigma2[i], M)
        mu, kap = ol.plain_index_params(prob, k[i])
        tol = 2e-4 * max(1.0, M ** 0.5 / 8)   # float32 sums of up to 16 terms that grow with the levels
        np.testing.assert_allclose(rows[i, :, :, 7], mu[:, 0::2], atol=tol)
        np.testing.assert_allclose(rows[i, :, :, 8], mu[:, 1::2], atol=tol)
        np.testing.assert_allclose(rows[i, :, :, :7], ol.features(prob, k[i], mu), atol=tol)
        np.testing.assert_allclose(rows[i, :, :, 9], kap, rtol=1e-6)
        assert np.all(rows[i, :, :, 10] == round(M ** 0.5)) and np.all(rows[i, :, :, 11] == 0)
