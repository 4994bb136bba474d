"""FP64 products on INT8 matrix cores at the edges of their kernels: residue
sums at the int32 limit, one to a few K slabs on the large tile, tile counts
that the XCD order does not divide, and the bytes of the widest integers."""
import numpy as np
import pytest

from test_gpu_ozaki import _run, _same, _want, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [128.0, 127.0, -127.0])
def test_residue_sums_at_the_int32_limit(torch_cuda, b):  # noqa: F811
    """128 has the residue -128 modulo 256: k = 131071 products of -128 with
    -128 or +-127 sum to just inside int32; the exact product is known."""
    k = 131071
    A, B = np.full((40, k), 128.0), np.full((k, 33), b)
    got = _run(torch_cuda, A, B, 0)
    assert np.array_equal(got, np.full((40, 33), 128.0 * b * k))


@pytest.mark.parametrize("m,n,k", [(1024, 1024, 1), (1024, 1281, 63), (1281, 1024, 65), (1300, 1100, 128),
                                   (1025, 1800, 192), (1024, 1024, 257)])
def test_few_slabs_on_the_large_tile(torch_cuda, m, n, k):  # noqa: F811
    g = np.random.default_rng(m + n + k)
    A, B = g.standard_normal((m, k)), g.standard_normal((k, n))
    got = _run(torch_cuda, A, B, 0, pad=1)
    rows = sorted({0, 1, 255, 256, 257, 511, 1023, m - 1} & set(range(m)))
    assert _same(np.ascontiguousarray(got[rows]), _want(A[rows], B, 0, None, 14, 0))


@pytest.mark.parametrize("moduli,beta", [(15, 53), (14, 47), (3, 0)])
def test_widest_integers(torch_cuda, moduli, beta):  # noqa: F811
    """Entries whose scaled integers are all ones, powers of two and their
    neighbours, with both signs."""
    g = np.random.default_rng(beta)
    k = 24
    e = g.integers(0, 53, size=(37, k))
    A = (np.ldexp(1.0, e) - g.integers(0, 2, size=e.shape)) * g.choice([-1.0, 1.0], size=e.shape)
    A[:, 0] = 2.0 ** 53 - 1
    e = g.integers(0, 53, size=(k, 21))
    B = (np.ldexp(1.0, e) - g.integers(0, 2, size=e.shape)) * g.choice([-1.0, 1.0], size=e.shape)
    B[0, :] = 2.0 ** 53 - 1
    got = _run(torch_cuda, A, B, 0, moduli=moduli, beta=beta)
    assert _same(got, _want(A, B, 0, None, moduli, beta))
