"""Autotuning a small plan, whose untuned classes run the spread kernels: never a slower choice, and its cache entries
apart from those of larger plans."""
import json

import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _plan(dm, nt, nr, M, n, C, T):
    b = W.make_batch(nt, nr, M, 20.0, n, seed=nt)
    H, y, s2 = dm.device_inputs(b.H, b.y, b.sigma2)
    return dm.Plan([(nt, nr, M)] * n, C, T, 5), (H.reshape(-1), y.reshape(-1), s2)


def _time(plan, args):
    import torch
    out, ms = [], []
    for _ in range(12):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        o = plan(*args)
        b.record()
        torch.cuda.synchronize()
        ms.append(a.elapsed_time(b))
    return float(np.median(ms[2:])), {k: v.cpu().numpy() for k, v in o.items()}


def _entries(path):
    return json.load(open(path))["entries"]


@pytest.mark.parametrize("nt,nr,M", [(64, 64, 64), (32, 32, 64), (16, 18, 16)])
def test_tuned_small_plan_is_not_slower(nt, nr, M, tmp_path):
    import paper_2407_06042_amd as dm
    cache = str(tmp_path / "tune.json")
    # a large plan of the same class first: its entry must not decide the small one's
    big, big_in = _plan(dm, nt, nr, M, 1100, 32, 20)
    big.autotune(*big_in, cache)
    assert [e["tile_config"] > 0 for e in _entries(cache)] == [True]
    plan, args = _plan(dm, nt, nr, M, 2, 32, 100)
    small_T20, args20 = _plan(dm, nt, nr, M, 2, 32, 20)
    small_T20.autotune(*args20, cache)      # the large plan's number of transitions
    t0, o0 = _time(plan, args)
    plan.autotune(*args, cache)
    t1, o1 = _time(plan, args)
    print("untuned %.3f ms, tuned %.3f ms: %s" % (t0, t1, _entries(cache)), flush=True)
    assert len(_entries(cache)) == 3
    # the layouts' own kernels take 1.6 to 2.6 times as long
    assert t1 < 1.3 * t0
    t20, _ = _time(small_T20, args20)
    t20_own, _ = _time(_plan(dm, nt, nr, M, 2, 32, 20)[0], args20)
    assert t20 < 1.3 * t20_own
    # another plan takes the choice from the cache
    again, args = _plan(dm, nt, nr, M, 2, 32, 100)
    again.autotune(*args, cache)
    assert len(_entries(cache)) == 3 and again.classes() == [dict(c, tuned_ms=d["tuned_ms"]) for c, d in zip(plan.classes(), again.classes())]
    np.testing.assert_allclose(again.classes()[0]["tuned_ms"], plan.classes()[0]["tuned_ms"], rtol=1e-4, atol=1e-6)
    t2, o2 = _time(again, args)
    assert t2 < 1.3 * t0
    for k in o0:   # (the spread kernels and their layouts give the same bits)
        np.testing.assert_array_equal(o1[k].view(np.uint8), o2[k].view(np.uint8), err_msg=k)
