"""Unnormalised FP32 powers of very small and large magnitudes, whose squares are
near the ends of the floats, against the FP64 form (needs an MI355X).

Tolerance: that of the FP32 form (test_gpu_mx.py), on the scale of the largest
power, and one unit of the smallest float, 1.4e-45."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402
from test_gpu_mx import ATOL, close  # noqa: E402
from test_gpu_parity import cuda, dev  # noqa: E402,F401

pytestmark = pytest.mark.gpu


# One object (shared tiles; parts of a long series), and a tile a wave
@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n_t,copies", [(300, 1), (3000, 1), (300, 450)])
@pytest.mark.parametrize("scale", [1e-19, 1e-18, 3e-16, 1e-10, 1.0, 1e10, 1e16])
def test_unnormalized_power(dev, method, n_t, copies, scale):
    t, y, _ = synth.sine_object(n_t, 31)
    dy = np.random.default_rng(8).uniform(0.03, 0.08, n_t)
    off = np.arange(copies + 1, dtype=np.int64) * n_t

    def call(form, c):
        return lsp.Periodogram(
            cuda(np.tile(t, c), dev), cuda(np.tile(y * scale, c), dev), 1.0, 12.0, 5000,
            offsets=None if c == 1 else cuda(off[:c + 1], dev, torch.int64), form=form,
            normalize=False, method=method, pgram_dtype=lsp.PGRAM_F64,
            dy=cuda(np.tile(dy, c), dev) if method == "generalized" else None)()

    got, ref = call(lsp.FORM_FP32P, copies), call(lsp.FORM_FP64, 1)
    row, want = got.pgram.cpu().numpy(), ref.pgram.cpu().numpy()[0]
    top = want.max()
    close(row / top, want[None] / top, f"{method} x{scale:g}", ATOL + 1.4e-45 / top)
    pk = got.peaks()
    assert np.all(want[pk["index"]] >= top * (1 - 2 * ATOL) - 3e-45)
