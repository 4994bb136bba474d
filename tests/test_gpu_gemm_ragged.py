"""Block products of sizes, leading dimensions and addresses that no 16-byte
vector divides: every edge of the vector width, of the 32/64/128 tiles and of
the K slab, against an FP64 reference within 4 (k + 2) u (|A| |B| + |C|)
elementwise (u of the product's type).  Padding around the operands is NaN: it
must neither reach a result nor be written."""
import numpy as np
import pytest

from test_gpu_leafspec import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(1, 5, 7), (2, 3, 1), (3, 1, 2), (4, 4, 3), (5, 9, 33), (31, 32, 31), (33, 31, 32), (63, 65, 64),
          (65, 63, 17), (129, 130, 15), (255, 257, 100), (513, 700, 47), (1537, 1001, 77), (1025, 1100, 33),
          (1793, 1795, 49), (2049, 1666, 16), (130, 4, 1), (4, 3000, 65)]


def _buf(torch, rows, cols, pad, off, dtype, g):
    """A column-major rows x cols view, leading dimension rows + pad, starting
    `off` elements into its allocation; NaN elsewhere."""
    ld = rows + pad
    flat = torch.full((off + ld * cols + 3,), float("nan"), dtype=dtype, device="cuda")
    v = flat[off:off + ld * cols].view(cols, ld)
    v[:, :rows] = torch.from_numpy(g.standard_normal((cols, rows))).to(dtype).cuda()
    return flat, v, ld


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("pad,off", [(0, 0), (1, 1), (3, 0)])
def test_ragged_product(torch_cuda, m, n, k, pad, off, dtype):  # noqa: F811
    import paper_1801_04723_amd as S
    torch = torch_cuda
    dt = torch.float64 if dtype == "fp64" else torch.float32
    u = 2.0 ** -53 if dtype == "fp64" else 2.0 ** -24
    g = np.random.default_rng(m + 3 * n + 7 * k + pad)
    fa, a, lda = _buf(torch, m, k, pad, off, dt, g)
    fb, b, ldb = _buf(torch, k, n, pad, off, dt, g)
    fc, c, ldc = _buf(torch, m, n, pad, off, dt, g)
    fd, d, ldd = _buf(torch, m, n, pad, off, dt, g)
    size = 8 if dtype == "fp64" else 4
    ptr = [f.data_ptr() + off * size for f in (fa, fb, fc, fd)]
    S.gemm_cm(m, n, k, -1.0, ptr[0], lda, ptr[1], ldb, 1.0, ptr[2], ldc, ptr[3], ldd, dtype=dtype)
    torch.cuda.synchronize()
    A, B, C = (x.double().cpu().numpy().T[:r] for x, r in ((a, m), (b, k), (c, m)))
    got = d.double().cpu().numpy().T
    ref = C - A @ B
    tol = 4 * (k + 2) * u * (np.abs(A) @ np.abs(B) + np.abs(C))
    assert np.all(np.abs(got[:m] - ref) <= tol)
    if pad:
        assert np.isnan(got[m:]).all()
