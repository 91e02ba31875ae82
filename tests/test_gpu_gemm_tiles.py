"""Every tile size of the BF16 product, at its edges (needs an MI355X).

Operands are whole numbers up to 2, so every sum is exact in FP32 and the
results must equal the whole-number product bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import mlp_ref  # noqa: E402
from paper_2105_04006_amd import learned  # noqa: E402

pytestmark = pytest.mark.gpu


def bits(a):
    return torch.as_tensor(mlp_ref.bf16_bits(a).view(np.int16), device="cuda:0")


# tiles of 128: 2 x 257 of them; of 64: 2 x 65; of 32: 2 x 2 and 1.  K: less
# than a step of 64, a whole number of steps, one to several steps and a rest.
@pytest.mark.parametrize("K", [40, 64, 136, 328])
@pytest.mark.parametrize("M,N", [(32776, 136), (32833, 136), (4104, 72), (4101, 72), (40, 40),
                                 (33, 40), (8, 8)])
def test_tiles_and_their_edges(M, N, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(M + 7 * K)
    A = rng.integers(-2, 3, (M, K)).astype(np.float32)
    B = rng.integers(-2, 3, (K, N)).astype(np.float32)
    bias = rng.integers(-9, 10, N).astype(np.float32)
    mask = rng.integers(-1, 2, (M, N)).astype(np.float32)
    ref = A @ B
    forms = [("X.W", bits(A), K, 1, bits(B), N, 1),
             ("dY.W^T", bits(A), K, 1, bits(np.ascontiguousarray(B.T)), 1, K)]
    if M % 8 == 0:
        forms.append(("X^T.dY", bits(np.ascontiguousarray(A.T)), 1, M, bits(B), N, 1))
    for name, a, sam, sak, b, sbk, sbn in forms:
        print(f"gemm {name} {M}x{K}x{N}", flush=True)
        Cf = torch.full((M + 1, N), 7.0, dtype=torch.float32, device="cuda:0")
        Cb = torch.full((M + 1, N), 7, dtype=torch.int16, device="cuda:0")
        learned.gemm(a, b, M, N, K, sam, sak, sbk, sbn, C=Cf, C_bf16=Cb)
        torch.cuda.synchronize()
        assert np.array_equal(Cf[:M].cpu().numpy(), ref)
        assert np.array_equal(mlp_ref.from_bf16_bits(Cb[:M].cpu().numpy().view(np.uint16)),
                              mlp_ref.bf16_round(ref))
        # nothing past the last row
        assert bool((Cf[M] == 7.0).all()) and bool((Cb[M] == 7).all())
        learned.gemm(a, b, M, N, K, sam, sak, sbk, sbn, C=Cf, mask=bits(mask), relu=True,
                     bias=torch.as_tensor(bias, device="cuda:0"))
        torch.cuda.synchronize()
        assert np.array_equal(Cf[:M].cpu().numpy(), np.maximum(ref + bias, 0.0) * (mask > 0))
