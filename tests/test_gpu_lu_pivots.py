"""Pivots of the LU leaf at the ends of the format: where a reciprocal is not a
normal number the multipliers are quotients all the same, so a tiny or huge
pivot that is not zero is no breakdown and spoils nothing but what it divides.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_lu import U, _dev, _host, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 16, 40, 64, 65, 128])
@pytest.mark.parametrize("at", ["first", "middle", "last"])
@pytest.mark.parametrize("piv", [1e-310, 2.0 ** -1074, -1e-309])
def test_subnormal_pivot_spoils_its_row_only(torch_cuda, L, at, piv):  # noqa: F811
    import paper_1801_04723_amd as S
    k = {"first": 0, "middle": L // 2, "last": L - 1}[at]
    A = np.diag(np.where(np.arange(L) == k, piv, 2.0))
    X = _host(S.invert_lu(_dev(torch_cuda, A), leaf=L))
    assert S.info() == oracle.lu_inv(A, L)[1] == 0
    keep = np.arange(L) != k
    assert not np.isfinite(X[k, k])
    assert np.array_equal(X[keep], np.diag(np.where(keep, 0.5, 0.0))[keep])


@pytest.mark.parametrize("L", [5, 40, 64, 128])
@pytest.mark.parametrize("scale", [-1024, -1014, -1010, 1005, 1013])
def test_scaled_matrices(torch_cuda, L, scale):  # noqa: F811
    """A = 2^scale B exactly, so X = 2^-scale B^-1.  What falls below the normal
    range on the way is rounded at 2^-1075 an operation, at most L 2^-53 of the
    smallest pivot (4 2^-1024), below the tolerance."""
    import paper_1801_04723_amd as S
    B = np.round(W.diag_dominant(L, seed=L) * 2.0 ** 20) * 2.0 ** -20
    A = np.ldexp(B, scale)
    X = _host(S.invert_lu(_dev(torch_cuda, A), leaf=L))
    assert S.info() == oracle.lu_inv(A, L)[1] == 0
    ref = oracle.lu_inv(B, L)[0]
    tol = max(1e-13, 100 * np.linalg.cond(B) * U) * np.linalg.norm(ref)
    assert np.linalg.norm(np.ldexp(X, scale) - ref) <= tol
