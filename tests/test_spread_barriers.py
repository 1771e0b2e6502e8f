"""The spread sampler's shared arrays are ordered by its barriers.

A wave may run up to one barrier ahead of another: between a wave's read of a shared array and any wave's
next write to it there has to be a barrier, as between a write and the reads of it.  The transition loop's
accesses and barriers are read off the source in order and followed over two transitions.  (The barrier that the
optional trace adds does not count.)
"""
import os
import re

import numpy as np
import pytest

import workloads as W
from tests.helpers import gpu_available, run_gpu

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_06042_amd", "csrc",
                   "sampler_spread.hpp")

# (pattern, access, array): the helpers' accesses as their definitions have them
EVENTS = [(r"__syncthreads\(\)", "barrier", ""), (r"\bput_levels\(", "write", "xbuf"), (r"\bgrad_at\(", "read", "xbuf"),
          (r"\bput\((\d)", "write", "term"), (r"\bget\((task|\d)", "read", "term"), (r"\bwords_end\(", "write", "wbuf"),
          (r"\btake_words\(", "read", "wbuf"), (r"\blub\[lane\]\s*=", "write", "lub"), (r"\blub\[lane\]\s*[^=\s]", "read", "lub"),
          (r"\bres\[[^\]]*\]\s*=", "write", "res"), (r"=\s*res\s*\+", "read", "res")]


def _block(text, at):
    """The braces' content from the first '{' at or after `at`, and its end."""
    i = text.index("{", at)
    depth, j = 0, i
    while True:
        depth += {"{": 1, "}": -1}.get(text[j], 0)
        j += 1
        if depth == 0:
            return text[i + 1:j - 1], j


def _loop_events():
    text = re.sub(r"//[^\n]*", "", open(SRC).read())
    loop, _ = _block(text, text.index("for (int t = 1; t <= a.T; ++t)"))
    at = loop.index("if (a.trace_hash)")
    loop = loop[:at] + loop[_block(loop, at)[1]:]
    ev = []
    for pat, kind, name in EVENTS:
        for m in re.finditer(pat, loop):
            names = [name]
            if name == "term":
                names = ["term0", "term1"] if m.group(1) == "task" else ["term" + m.group(1)]
            ev += [(m.start(), kind, n) for n in names]
    return [(k, n) for _, k, n in sorted(ev)]


def test_every_shared_array_is_ordered():
    one = _loop_events()
    arrays = sorted({n for _, n in one if n})
    assert arrays == ["lub", "res"] + ["term%d" % i for i in range(6)] + ["wbuf", "xbuf"]
    assert sum(k == "barrier" for k, _ in one) == 3
    ev = one + one
    for name in arrays:
        kinds = {k for k, n in one if n == name}
        assert kinds == {"read", "write"}, (name, kinds)
        last = None
        for kind, n in ev:
            if kind == "barrier":
                last = None
            elif n == name:
                assert last in (None, kind), "%s: %s after %s without a barrier" % (name, kind, last)
                last = kind


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("nt,nr,M,n,C,layout", [(64, 64, 64, 128, 32, 8), (32, 32, 64, 512, 32, 10), (16, 16, 256, 768, 32, 1)])
def test_full_grids_without_a_trace(nt, nr, M, n, C, layout):
    """The largest launches that are spread, untraced: bit for bit the layout kernel's chains."""
    outs = ("symbols", "best_energy", "final_state", "accept_count")
    batch = W.make_batch(nt, nr, M, 18.0, n, seed=nt)
    _, a = run_gpu(batch, C, 100, 5, outputs=outs, trace=False)
    _, b = run_gpu(batch, C, 100, 5, outputs=outs, trace=False, tile_config=layout)
    for k in outs:
        np.testing.assert_array_equal(a[k].view(np.uint8), b[k].view(np.uint8), err_msg=k)
