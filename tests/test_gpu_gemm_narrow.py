"""Products with few rows or columns: the tile chosen for them may not show in
the result (needs an MI355X).

A product adds its k in the same blocks whatever the tile, so it is bit-equal to
the same numbers as part of a larger one."""
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import learned  # noqa: E402
from test_gpu_parity import dev  # noqa: E402,F401

pytestmark = pytest.mark.gpu


def bits(dev, *shape):
    g = torch.Generator(device=dev)
    g.manual_seed(sum(shape))
    return torch.randn(shape, generator=g, device=dev).to(torch.bfloat16).view(torch.int16)


@pytest.mark.parametrize("N", [1, 8, 32, 33, 64, 65])
@pytest.mark.parametrize("M,K", [(70_000, 64), (70_001, 72), (9000, 200), (130, 1088)])
def test_narrow_products(dev, M, K, N):
    A, B = bits(dev, M, K), bits(dev, K, 192)
    wide = torch.empty(M, 192, device=dev)
    learned.gemm(A, B, M, 192, K, K, 1, 192, 1, C=wide)
    some = B[:, :(N + 7) // 8 * 8].contiguous()  # rows of a multiple of 16 bytes
    C = torch.empty(M, N, device=dev)
    learned.gemm(A, some, M, N, K, K, 1, some.shape[1], 1, C=C)
    # and with the few ones as rows: C' = B' A'
    T = torch.empty(N, M, device=dev)
    learned.gemm(some, A, N, M, K, 1, some.shape[1], 1, K, C=T)
    torch.cuda.synchronize()
    assert torch.equal(C, wide[:, :N])
    assert torch.equal(T.T, C)
    ref = A.view(torch.bfloat16).double() @ some.view(torch.bfloat16).double()[:, :N]
    assert torch.all((C - ref).abs() <= 2.0 ** -23 * K * ref.abs().max())
