"""A plan's workspace holds every layout that its autotuner tries, not the default ones alone."""
import ctypes

import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

C, T = 32, 4
CLASSES = [(64, 64, 64, 5), (32, 32, 16, 7), (100, 110, 4, 2), (9, 12, 256, 6)]


def _largest(dm, nt, nr, M, n, precision):
    size = dm.lib().dmala_workspace_size
    return max(size(n, nt, nr, M, ctypes.byref(dm.make_params(C, T, 5, precision, tile_config=tc))) for tc in range(11))


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16", "fp64"])
def test_workspace_covers_every_layout(precision):
    import paper_2407_06042_amd as dm
    cls = [c for c in CLASSES if precision != "fp64" or c[0] <= 32]
    for nt, nr, M, n in cls:
        assert dm.Plan([(nt, nr, M)] * n, C, T, 5, precision).ws_bytes >= _largest(dm, nt, nr, M, n, precision)
    mixed = dm.Plan([c[:3] for c in cls for _ in range(c[3])], C, T, 5, precision)
    assert mixed.ws_bytes >= sum(_largest(dm, *c, precision) for c in cls)


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_autotuning_stays_inside_the_workspace(precision):
    import torch
    import paper_2407_06042_amd as dm
    need = sum(_largest(dm, *c, precision) for c in CLASSES)
    parts = [[], [], []]
    for nt, nr, M, n in CLASSES:
        b = W.make_batch(nt, nr, M, 20.0, n, seed=nt)
        for p, v in zip(parts, dm.device_inputs(b.H, b.y, b.sigma2, precision)):
            p.append(v.reshape(-1))
    args = [torch.cat(p) for p in parts]
    plan = dm.Plan([c[:3] for c in CLASSES for _ in range(c[3])], C, T, 5, precision)
    # the workspace at the head of a buffer with room for all layouts many times over
    buf = torch.full((4 * max(need, plan.ws_bytes) + 512,), 0xA5, dtype=torch.uint8, device="cuda")
    plan.ws = buf
    tail = (-buf.data_ptr()) % 256 + plan.ws_bytes
    plan.autotune(*args)
    tuned = plan(*args)["final_state"].cpu().numpy()
    torch.cuda.synchronize()
    assert bool((buf[tail:] == 0xA5).all())
    # a different layout changes only summation order: nearly all chains unchanged
    own = dm.Plan(plan.shapes, C, T, 5, precision)(*args)["final_state"].cpu().numpy()
    assert np.mean(tuned == own) > 0.9
