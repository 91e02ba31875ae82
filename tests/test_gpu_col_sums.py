"""Column sums of wide matrices: the columns per workgroup may not show in the
result (needs an MI355X).

They add the same 16 phases either way, so they are bit-equal to those of a part
of the columns."""
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import learned, lsp  # noqa: E402
from test_gpu_parity import dev  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 15, 16, 17, 31, 32, 33, 127, 129, 1000])
@pytest.mark.parametrize("c", [16_383, 16_384, 16_385, 20_001])
def test_column_sums_of_wide_matrices(dev, n, c):
    g = torch.Generator(device=dev)
    g.manual_seed(n + c)
    x = torch.randn(n, c, generator=g, device=dev)
    out = torch.full((c,), 7.0, device=dev)

    def sums(x, out):
        learned._ok(lsp.lib().lsp_col_sums(learned._p(x), x.shape[0], x.shape[1],
                                           learned._p(out), learned._s()), "lsp_col_sums")

    sums(x, out)
    torch.cuda.synchronize()
    for a in (0, 64, c - 100):
        part = torch.empty(100, device=dev)
        own = x[:, a:a + 100].contiguous()
        sums(own, part)
        torch.cuda.synchronize()
        assert torch.equal(out[a:a + 100], part)
    assert torch.allclose(out.double(), x.double().sum(0), atol=1e-6 * max(1, n))
