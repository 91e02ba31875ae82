"""Statistics of long series, around the number of observations that a thread
loads together (needs an MI355X).

The normalised power is the unnormalised one times 2 / S, S = sum w (y - ybar)^2
in the caller's weights, so their ratio shows S.  S is a sum of n non-negative
FP64 terms, each from a mean of n terms that moves S only in second order, so it
is within (n + 10) u of the exact sum relatively, and so is numpy's; both powers
are rounded a few times more: 4 (n + 20) u in all, u = 2^-53."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n", [255, 257, 1792, 2047, 2048, 2049, 4096, 4097, 5000])
def test_long_series(n, method):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n)
    t = rng.uniform(0.0, 900.0, n)
    y = rng.normal(12.0, 0.3, n)
    dy = rng.uniform(0.03, 0.3, n) if method == "generalized" else None
    dev = lambda a: None if a is None else torch.as_tensor(a, device="cuda:0")  # noqa: E731

    def call(yy, normalize, e):
        p = lsp.Periodogram(dev(t), dev(yy), 1.0, 2.0, 600, form=lsp.FORM_FP64, method=method,
                            dy=dev(e), normalize=normalize, pgram_dtype=lsp.PGRAM_F64)()
        torch.cuda.synchronize()
        return p.pgram.cpu().numpy().ravel(), p.peaks()

    print(f"statistics n={n} {method}", flush=True)
    w = np.ones(n) if dy is None else 1.0 / dy ** 2
    mean = np.sum(w * y) / np.sum(w)
    s = np.sum(w * (y - mean) ** 2)
    norm, raw = call(y, True, dy)[0], call(y, False, dy)[0]
    assert np.all(np.abs(norm / raw * s / 2.0 - 1.0) <= 4 * (n + 20) * 2.0 ** -53)
    for at in (0, n // 2, n - 1):  # one bad value anywhere is found
        bad = y.copy()
        bad[at] = np.inf
        assert call(bad, True, dy)[1]["status"][0] == lsp.OBJ_NONFINITE
        if dy is not None:
            e = dy.copy()
            e[at] = 0.0
            assert call(y, True, e)[1]["status"][0] == lsp.OBJ_NONFINITE
