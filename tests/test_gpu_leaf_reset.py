"""Inversions that are one whole leaf: its kernel resets the status block.

A failure is reported by its own call only, with speculation on and off, and a
larger inversion or a residual between the calls finds the block as it needs it.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_leafspec import _both, _dev, _same_bits, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 64, 65, 128])
@pytest.mark.parametrize("entry", ["invert", "invert_spd"])
def test_status_of_each_call_is_its_own(torch_cuda, L, entry):  # noqa: F811
    import paper_1801_04723_amd as S
    f = getattr(S, entry)
    good = _dev(torch_cuda, W.spd_gram(L, seed=L) if hasattr(W, "spd_gram") else W.diag_dominant(L, seed=L))
    bad = np.asfortranarray(np.eye(L))
    bad[L // 2, L // 2] = 0.0
    bad = _dev(torch_cuda, bad)
    big = _dev(torch_cuda, W.diag_dominant(300, seed=2))
    _, s0, _, s1 = _both(lambda: f(bad, leaf=L))
    assert s0 == s1 == L // 2 + 1
    x0, s0, x1, s1 = _both(lambda: f(good, leaf=L))
    assert s0 == s1 == 0 and _same_bits(x0, x1)
    x, s0, y, s1 = _both(lambda: S.invert(big, leaf=64))
    assert s0 == s1 == 0 and _same_bits(x, y)
    x0, s0, x1, s1 = _both(lambda: f(bad, leaf=L))
    assert s0 == s1 == L // 2 + 1
    x = f(good, leaf=L)
    assert S.residual(good, x) < 1e-15 and S.info() == 0
