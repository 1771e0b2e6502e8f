"""The learned proposal beyond 64 antennas: 4-QAM evaluates the network one antenna group after another (the other
alphabets two at a time)."""
import numpy as np
import pytest

from tests.helpers import gpu_available
from tests.test_gpu_learned import test_mixture_chains_follow_the_oracle as _follow

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("nt", [65, 100])
def test_four_qam_follows_the_oracle(nt):
    _follow(nt, 4, 0.2, 0)


def _time(n, nt, M):
    """Median time of the sampler, 32 chains, 20 transitions."""
    import torch
    import paper_2407_06042_amd as dm
    g = torch.Generator(device="cuda").manual_seed(1)
    H = torch.randn(n, nt, nt, dtype=torch.complex64, device="cuda", generator=g) / nt ** 0.5
    y = torch.randn(n, nt, dtype=torch.complex64, device="cuda", generator=g)
    s2 = torch.full((n,), 0.1, device="cuda")
    w = torch.randn(dm.MLP_PARAMS, device="cuda", generator=g) * 0.1
    d = dm.Detector(n, nt, nt, M, 32, 20, 1, proposal="learned", mlp_weights=w, mix_eps=0.3)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in ev:
        e.record()
    ms = []
    for _ in range(9):
        d(H, y, s2, events=[e.cuda_event for e in ev])
        torch.cuda.synchronize()
        ms.append(ev[1].elapsed_time(ev[2]))
    return float(np.median(ms[2:]))


@pytest.mark.parametrize("n,nt", [(375, 85), (300, 128)])
def test_four_qam_takes_less_than_sixteen(n, nt):
    """Fewer levels to weigh, else the same work (two groups at a time 1.03 and 1.06 times as long as 16-QAM)."""
    a, b = min(_time(n, nt, 4) for _ in range(2)), min(_time(n, nt, 16) for _ in range(2))
    print("%.3f ms, 16-QAM %.3f" % (a, b), flush=True)
    assert a < 0.97 * b
