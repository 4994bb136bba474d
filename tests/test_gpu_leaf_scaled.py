"""Leaves whose pivots lie far from 1: eliminated without the search as others
are, with the search's bits, over the whole range of the format.
"""
import os

import numpy as np
import pytest

import workloads as W
from test_gpu_leafblocks import _compare
from test_gpu_leafspec import _dev, _same_bits, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

ORDERS = (16, 20, 64, 100, 128, 150, 320, 512)


def _ms(torch, L, a, reps=20):
    import paper_1801_04723_amd as S
    x = torch.empty_like(a)
    best = float("inf")
    for _ in range(5):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(reps):
            S.invert(a, leaf=L, out=x)
        t1.record()
        torch.cuda.synchronize()
        best = min(best, t0.elapsed_time(t1) / reps)
    return best


@pytest.mark.parametrize("L", [64, 128, 320])
@pytest.mark.parametrize("scale", [-600, 600])
def test_scaled_leaves_skip_the_search(torch_cuda, L, scale):  # noqa: F811
    """A fourth of the search's time at least is saved, as it is at scale 0."""
    a = _dev(torch_cuda, np.ldexp(W.diag_dominant(L, seed=L), scale))
    _ms(torch_cuda, L, a)
    fast = _ms(torch_cuda, L, a)
    os.environ["SPIN_NO_SPEC"] = "1"
    try:
        search = _ms(torch_cuda, L, a)
    finally:
        del os.environ["SPIN_NO_SPEC"]
    assert fast <= 0.75 * search


@pytest.mark.parametrize("L", ORDERS)
@pytest.mark.parametrize("scale", [-1060, -1027, -1010, -520, -404, 396, 505, 1010])
def test_scaled_leaves_equal_the_search(torch_cuda, L, scale):  # noqa: F811
    x0, x1, _ = _compare(torch_cuda, np.ldexp(W.diag_dominant(L, seed=L + 1), scale), L)
    assert _same_bits(x0, x1)


@pytest.mark.parametrize("L", ORDERS)
@pytest.mark.parametrize("step", [-1900, -300, 300, 1900])
def test_graded_leaves_equal_the_search(torch_cuda, L, step):  # noqa: F811
    """Rows and columns scaled from 1 down (or up) to 2^(step / 2): pivots from
    both sides of the division's range in one leaf, no row exchanges."""
    e = np.arange(L) * (step // 4) // L
    A = np.ldexp(W.diag_dominant(L, seed=L), e[:, None] + e[None, :])
    if step > 0:
        A = A[::-1, ::-1].copy()
    x0, x1, st = _compare(torch_cuda, A, L)
    assert st == 0 and _same_bits(x0, x1)


@pytest.mark.parametrize("L", ORDERS)
@pytest.mark.parametrize("at", ["first", "fourth", "middle", "last"])
@pytest.mark.parametrize("piv", [2.0 ** -1074, -2.0 ** -1024, 2.0 ** 1023])
def test_one_far_pivot_equals_the_search(torch_cuda, L, at, piv):  # noqa: F811
    """Also where its reciprocal overflows (the infinities stay where the search
    puts them) with entries left of it that it divides."""
    k = {"first": 0, "fourth": 3, "middle": L // 2, "last": L - 1}[at]
    A = np.eye(L) * 2.0
    A[k, k] = piv
    A[k, :k] = 0.5
    x0, x1, _ = _compare(torch_cuda, A, L)
    assert _same_bits(x0, x1)


@pytest.mark.parametrize("L", ORDERS)
def test_far_pivot_behind_a_plain_diagonal(torch_cuda, L):  # noqa: F811
    A = np.eye(L)
    A[1, 0], A[0, 1], A[1, 1] = 1.0, 2.0 ** 600, 2.0 ** 300
    x0, x1, st = _compare(torch_cuda, A, L)
    assert st == 0 and _same_bits(x0, x1)
