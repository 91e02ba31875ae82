"""The two statistics kernels (observations one by one, or eight a thread in
flight for calls of 2,048 points an object and more) give the same bits: an
object's powers from the plain FP64 kernel do not depend on the objects beside
it (needs an MI355X)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402
from test_gpu_parity import cuda, dev  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n_t", [1, 40, 2047, 2048, 2049, 5000])
def test_same_statistics_in_any_batch(dev, method, n_t):

    def powers(sizes):
        series = [(t, y) for t, y, _ in (synth.sine_object(n, n) for n in sizes)]
        off, t, y = synth.pack(series)
        dy = np.concatenate([np.random.default_rng(n).uniform(0.03, 0.08, n) for n in sizes])
        p = lsp.Periodogram(cuda(t, dev), cuda(y, dev), 1.0, 12.0, 300, k=2,
                            offsets=cuda(off, dev, torch.int64), form=lsp.FORM_FP64,
                            method=method,
                            dy=cuda(dy, dev) if method == "generalized" else None,
                            pgram_dtype=lsp.PGRAM_F64)()
        return p.pgram.cpu().numpy(), p.peaks()

    short, ps = powers([n_t, 10, 10, 10, 10, 10])
    long_, pl = powers([n_t, 9000, 9000, 9000])
    assert np.array_equal(short[0], long_[0], equal_nan=True)
    assert ps[0].tobytes() == pl[0].tobytes()
