"""Which calls are replayed as graphs, told by the host's time of a repeated
call: a graph's launch takes it much less than the call's own launches, of which
a call can have many though its schedule has one or a few steps.
"""
import ctypes
import os
import time

import numpy as np
import pytest

import workloads as W
from test_gpu_leafspec import _dev, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def _host_us(torch, fn, reps=40):
    """Least host time of a call to fn alone, over its third and later calls."""
    for _ in range(3):
        fn()
    best = float("inf")
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        fn()
        best = min(best, time.perf_counter() - t0)
    torch.cuda.synchronize()
    return best * 1e6


def _direct_us(torch, fn):
    os.environ["SPIN_NO_GRAPH"] = "1"
    try:
        return _host_us(torch, fn)
    finally:
        del os.environ["SPIN_NO_GRAPH"]


@pytest.mark.parametrize("call,n,leaf", [("invert", 512, 512), ("invert", 600, 600), ("spd", 512, 256),
                                         ("fp32", 512, 512), ("fp32_int8", 64, 64), ("fp32_int8", 256, 128)])
def test_calls_of_many_launches_are_replayed(torch_cuda, call, n, leaf):  # noqa: F811
    import paper_1801_04723_amd as S
    a = _dev(torch_cuda, W.spd_gram(n, seed=n))
    x = torch_cuda.empty_like(a)
    fn = {"invert": lambda: S.invert(a, leaf=leaf, out=x), "spd": lambda: S.invert_spd(a, leaf=leaf, out=x)}.get(
        call, lambda: S.invert_mixed(a, leaf=leaf, mode=call, ns_steps=2, out=x))
    assert _host_us(torch_cuda, fn) <= 0.75 * _direct_us(torch_cuda, fn)


@pytest.mark.parametrize("L", [1, 64, 128, 129, 192, 256, 257, 320, 512, 513, 1024])
@pytest.mark.parametrize("mode", ["fp64", "fp32"])
def test_launch_count_of_a_leaf(torch_cuda, L, mode):  # noqa: F811
    """The count that the rule uses against the launches of a traced call."""
    import paper_1801_04723_amd as S
    count = S.lib()["_ZN4spin13leaf_launchesElNS_5DTypeE"]
    count.restype, count.argtypes = ctypes.c_int64, (ctypes.c_int64, ctypes.c_int)
    a = _dev(torch_cuda, W.diag_dominant(L, seed=L))
    S.release()
    S.trace_enable(True)
    try:
        if mode == "fp64":
            S.invert(a, leaf=L)
        else:
            S.invert_mixed(a, leaf=L, mode="fp32", ns_steps=0)
        torch_cuda.cuda.synchronize()
        recs = S.trace_collect()
    finally:
        S.trace_enable(False)
    assert len(recs) == count(L, 0 if mode == "fp64" else 1)
