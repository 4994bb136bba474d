"""Small products whose slabs are loaded several steps ahead.

Integer operands whose products and sums are exact in FP32 and FP64: the result
is the exact one at every number of slabs around the four that are in flight.
"""
import pytest

from test_gpu_leafspec import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["fp64", "fp32"])
@pytest.mark.parametrize("m,n,slabs", [(64, 32, 7), (64, 32, 8), (96, 80, 9), (256, 33, 10), (32, 100, 11),
                                       (128, 128, 12), (60, 70, 13), (64, 64, 31), (4, 1, 16)])
def test_exact_at_each_slab_count(torch_cuda, mode, m, n, slabs):  # noqa: F811
    torch = torch_cuda
    import paper_1801_04723_amd as S
    dt = torch.float64 if mode == "fp64" else torch.float32
    k = 32 * slabs
    g = torch.Generator(device="cuda").manual_seed(k + m)
    a = torch.randint(-30, 31, (k, m), device="cuda", generator=g).to(dt)
    b = torch.randint(-30, 31, (n, k), device="cuda", generator=g).to(dt)
    c = torch.randint(-30, 31, (n, m), device="cuda", generator=g).to(dt)
    d = torch.empty(n, m, device="cuda", dtype=dt)
    S.gemm_cm(m, n, k, -1.0, a, m, b, k, 1.0, c, m, d, m, dtype=mode)
    want = c.cpu().double() - b.cpu().double() @ a.cpu().double()  # |sums| < 2^20
    assert torch.equal(d.cpu().double(), want)


@pytest.mark.parametrize("mode", ["fp64", "fp32"])
@pytest.mark.parametrize("m,n,slabs", [(768, 768, 3), (768, 700, 4), (764, 768, 5), (1024, 512, 6), (512, 1023, 9)])
def test_exact_on_64_tiles(torch_cuda, mode, m, n, slabs):  # noqa: F811
    test_exact_at_each_slab_count(torch_cuda, mode, m, n, slabs)


@pytest.mark.parametrize("mode", ["fp64", "fp32"])
@pytest.mark.parametrize("m,n,k", [(33, 31, 31), (63, 65, 255), (61, 40, 257), (125, 7, 287), (5, 90, 321),
                                   (767, 769, 95), (769, 767, 129), (1023, 511, 161), (765, 770, 1)])
def test_exact_with_a_tail_slab(torch_cuda, mode, m, n, k):  # noqa: F811
    torch = torch_cuda
    import paper_1801_04723_amd as S
    dt = torch.float64 if mode == "fp64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(k + m)
    a = torch.randint(-30, 31, (k, m + 1), device="cuda", generator=g).to(dt)
    b = torch.randint(-30, 31, (n, k + 2), device="cuda", generator=g).to(dt)
    d = torch.empty(n, m, device="cuda", dtype=dt)
    S.gemm_cm(m, n, k, 1.0, a, m + 1, b, k + 2, 0.0, None, m, d, m, dtype=mode)
    want = b.cpu().double()[:, :k] @ a.cpu().double()[:, :m]
    assert torch.equal(d.cpu().double(), want)
