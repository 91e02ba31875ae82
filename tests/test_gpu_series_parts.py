"""One long series on a narrow grid: its observations split over workgroups whose
sums are added by a kernel of their own (needs an MI355X).  Against the vector
kernels (an explicit k_per_lane), with the FP32 forms' bound (test_gpu_mx.py)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402
from test_gpu_mx import ATOL, close, peak_near  # noqa: E402
from test_gpu_parity import cuda, dev  # noqa: E402,F401

pytestmark = pytest.mark.gpu


def series(dev, t, y, dy, lo, hi, n_f, method, **kw):
    return lsp.Periodogram(cuda(t, dev), cuda(y, dev), lo, hi, n_f, form=lsp.FORM_FP32P,
                           pgram_dtype=lsp.PGRAM_F64, method=method,
                           dy=cuda(dy, dev) if method == "generalized" else None, **kw)


# Around the first split (1,024 points), parts that are not whole slices, the
# most parts (64), and more tiles than parts
@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n_t", [1023, 1024, 1025, 1537, 4099, 40_003])
@pytest.mark.parametrize("n_f", [1, 1025, 2049, 20_000, 130_001])
def test_parts(dev, method, n_t, n_f):
    t, y, _ = synth.sine_object(n_t, n_t)
    dy = np.random.default_rng(n_t).uniform(0.03, 0.08, n_t)
    args = (dev, t, y, dy, 0.0, 12.0, n_f, method)  # from f = 0, the FP64 fix-up's
    got, ref = series(*args)(), series(*args, k=16)()
    row, want = got.pgram.cpu().numpy(), ref.pgram.cpu().numpy()
    close(row, want, f"{method} n_t={n_t} n_f={n_f}", 2 * ATOL)
    pk, rk = got.peaks(), ref.peaks()
    if rk["index"][0] < 0:  # one bin, f = 0, no power: no peak in either
        assert pk["index"][0] < 0 and row.max() == 0.0
        return
    assert pk["power"][0] == row[0, pk["index"][0]] == row.max()
    assert peak_near(want[0], pk["index"][0], 2 * ATOL)


@pytest.mark.parametrize("method", ["standard", "generalized"])
def test_parts_statuses_and_replays(dev, method):
    rng = np.random.default_rng(3)
    n_t, n_f = 5000, 6001
    t = np.arange(n_t, dtype=np.float64)  # f = 0, 1/2, 1: a vanishing regressor
    y, dy = rng.normal(size=n_t), rng.uniform(0.03, 0.08, n_t)
    call = series(dev, t, y, dy, 0.0, 1.5, n_f, method)
    plain = series(dev, t, y, dy, 0.0, 1.5, n_f, method, k=16)
    plan = lsp.Plan(call)
    for turn, fill in ((0, None), (1, np.nan), (2, 0.0), (3, None)):
        now = y.copy()
        if turn == 1:
            now[3333] = np.nan
        if turn == 2:
            now[:] = 0.25
        for c in (call, plain):
            c.y.copy_(cuda(now, dev))
        plain()
        torch.cuda.synchronize()
        want, status = plain.pgram.cpu().numpy(), plain.peaks()["status"][0]
        for run in (call, plan, plan):
            call.pgram.fill_(-5.0)
            run()
            torch.cuda.synchronize()
            row, pk = call.pgram.cpu().numpy(), call.peaks()
            assert pk["status"][0] == status
            if fill is None:
                close(row, want, f"{method} turn {turn}", 2 * ATOL)
                assert pk["power"][0] == row[0, pk["index"][0]] == row.max()
            else:
                assert pk["index"][0] == -1
                assert np.all(np.isnan(row) if np.isnan(fill) else row == fill)
