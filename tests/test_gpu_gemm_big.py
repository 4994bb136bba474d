"""The 256 x 256 tiles of the BF16 and bf16x3 products.

They take every element through the operations of the smaller tiles in the
same order, so a product that they compute equals, bit for bit, the same
product computed in column strips too narrow for them: at sizes that are no
multiple of the tile or of the 32-deep slab, with padded leading dimensions and
with each part of the epilogue.
"""
import pytest

from test_gpu_leafspec import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["bf16", "bf16x3"])
@pytest.mark.parametrize("m,n,k,pad", [(2560, 4096, 512, 0), (2564, 4092, 516, 4), (4096, 4096, 540, 8),
                                       (3332, 3329, 1056, 0), (256, 41000, 512, 0)])
def test_big_tiles_equal_small_tiles(torch_cuda, mode, m, n, k, pad):  # noqa: F811
    torch = torch_cuda
    import paper_1801_04723_amd as S
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    lda, ldb, ldd = m + pad, k + pad, m + pad + 1
    a = torch.randn(k, lda, device="cuda", generator=g)
    b = torch.randn(n, ldb, device="cuda", generator=g)
    c = torch.randn(n, ldd, device="cuda", generator=g)
    for alpha, beta, eye in ((1.0, 0.0, False), (-1.0, 1.0, True)):
        d = torch.zeros(n, ldd, device="cuda")
        S.gemm_cm(m, n, k, alpha, a, lda, b, ldb, beta, c, ldd, d, ldd, add_identity=eye, dtype=mode)
        e = torch.zeros(n, ldd, device="cuda")
        for j in range(0, n, 512):
            w = min(512, n - j)
            S.gemm_cm(m, w, k, alpha, a, lda, b[j:], ldb, beta, c[j:], ldd, e[j:], ldd, dtype=mode)
        if eye:  # the strips off the diagonal have no identity of their own
            i = torch.arange(min(m, n), device="cuda")
            d64 = e[i, i].double() + 1.0
            near = (d[i, i].double() - d64).abs()
            # one rounding of value + 1 in place of two
            assert bool((near <= 2.0 ** -23 * (d64.abs() + 2.0)).all())
            d[i, i] = e[i, i]
        assert torch.equal(d, e)
        assert bool((d[:, m:] == 0).all())
