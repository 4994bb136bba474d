"""Products with triangular operands: the k ranges in which a tile meets only
zeros are left out, so the result is the whole product's bit for bit (a sum that
starts from 0 and adds zeros is the sum without them; only the sign of a zero sum
may differ), on the vector, ragged and guarded kernels and at every tile.
"""
import ctypes

import pytest

from test_gpu_leafspec import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

A_LOWER, A_UPPER, B_LOWER, B_UPPER = 1, 2, 4, 8


class Prob(ctypes.Structure):
    """GemmProb of the library."""
    _fields_ = ([(f, ctypes.c_void_p) for f in ("A", "B", "C0", "D")]
                + [(f, ctypes.c_int64) for f in ("lda", "ldb", "ldc", "ldd")]
                + [(f, ctypes.c_int32) for f in ("m", "n", "k", "add_identity")]
                + [("alpha", ctypes.c_double), ("beta", ctypes.c_double),
                   ("lower", ctypes.c_int16), ("tri", ctypes.c_int16), ("lddt", ctypes.c_int32),
                   ("DT", ctypes.c_void_p)])


@pytest.mark.parametrize("tri", [A_LOWER, A_UPPER, B_LOWER, B_UPPER, A_UPPER | B_LOWER])
@pytest.mark.parametrize("h,other", [(1, 64), (3, 5), (64, 65), (65, 64), (96, 200), (128, 1), (129, 65),
                                     (193, 64), (512, 512), (1000, 999), (1536, 2048), (1801, 1777)])
def test_skipped_triangles(torch_cuda, tri, h, other):  # noqa: F811
    torch = torch_cuda
    import paper_1801_04723_amd as S
    launch = S.lib()["_ZN4spin11gemm_launchEPKNS_8GemmProbEiNS_5DTypeEP12ihipStream_tPNS_10LaunchInfoE"]
    launch.restype = ctypes.c_int
    launch.argtypes = [ctypes.POINTER(Prob), ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    assert ctypes.sizeof(Prob) == 112
    on_a, on_b = tri & 3, tri & 12
    m, k, n = (h if on_a else other), h, (h if on_b else other)
    g = torch.Generator(device="cuda").manual_seed(h + other)
    a = torch.randn(m, k, dtype=torch.float64, device="cuda", generator=g)
    b = torch.randn(k, n, dtype=torch.float64, device="cuda", generator=g)
    a = {0: a, A_LOWER: a.tril(), A_UPPER: a.triu()}[on_a].t().contiguous()  # column-major
    b = {0: b, B_LOWER: b.tril(), B_UPPER: b.triu()}[on_b].t().contiguous()
    out = []
    for t in (tri, 0):
        d = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
        p = Prob(a.data_ptr(), b.data_ptr(), None, d.data_ptr(), m, k, 1, m, m, n, k, 0, -1.0, 0.0, 0, t, 0, None)
        assert launch(ctypes.byref(p), 1, 0, torch.cuda.current_stream().cuda_stream, None) == 0
        out.append(d)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("kind,n,leaf", [("dd", 129, 64), ("dd", 193, 64), ("spd", 1001, 100), ("dd", 387, 128)])
def test_odd_orders(torch_cuda, kind, n, leaf):  # noqa: F811
    """Orders whose last block is a single row, or of odd size."""
    from test_gpu_lu import test_invert_lu_parity
    test_invert_lu_parity(torch_cuda, kind, n, leaf)
