"""The FP64 form's matrix-core sums (every tuning field left to the library)
against the plain FP64 kernel (an explicit k_per_lane) and the oracle (needs an
MI355X).

Both evaluate the grid's rounded frequencies in FP64, so both are held to the
FP64 form's bound, |dP| <= 1e-9 max(P, 1e-3) (the generalized form's moment
matrix adds 1e-14 kappa^2, its condition), and to twice that of each other.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402
from test_gpu_gen import moment_condition  # noqa: E402
from test_gpu_parity import assert_fp64_close, cuda, dev, oracle, run_batch, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu


def near(got, ref, what, kappa2=0.0):
    both_nan = np.isnan(got) & np.isnan(ref)
    err = np.where(both_nan, 0.0, np.abs(got - ref))
    tol = 2.0 * (1e-9 + 1e-14 * kappa2) * np.maximum(np.abs(np.nan_to_num(ref)), 1e-3)
    say(f"    {what}: worst {np.max(err / tol):.3g} of the bound")
    assert np.all(err <= tol), what


def call(dev, off, t, y, dy, lo, hi, n_f, k, method, **kw):
    p = lsp.Periodogram(cuda(t, dev), cuda(y, dev), lo, hi, n_f, form=lsp.FORM_FP64,
                        offsets=None if off is None else cuda(off, dev, torch.int64), k=k,
                        pgram_dtype=lsp.PGRAM_F64, method=method,
                        dy=cuda(dy, dev) if method == "generalized" else None, **kw)()
    return p.pgram.cpu().numpy(), p.peaks()


# Around a block (32 bins), a wave tile (512) and a workgroup's four; around a
# matrix step (4 observations), eight of them, and a staging pass (256); 300
# copies of the object take the one-tile-per-wave kernel, two the shared one
@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n_f", [1, 31, 33, 511, 513, 2047, 2049, 5000])
@pytest.mark.parametrize("n_t", [8, 31, 32, 33, 255, 257, 530])
def test_sizes(dev, method, n_f, n_t):
    rng = np.random.default_rng(n_t)
    t, y, _ = synth.sine_object(n_t, 3000 + n_t)
    dy = rng.uniform(0.03, 0.08, n_t)
    freqs = 1.0 + 11.0 / n_f * np.arange(n_f)
    k2 = moment_condition(t, dy, freqs) if method == "generalized" else 0.0
    ref, rk = call(dev, None, t, y, dy, 1.0, 12.0, n_f, 2, method)
    for c in (1, 2, 600 if n_f < 600 else 300):
        off = np.arange(c + 1, dtype=np.int64) * n_t
        got, pk = call(dev, None if c == 1 else off, np.tile(t, c), np.tile(y, c), np.tile(dy, c),
                       1.0, 12.0, n_f, 0, method)
        assert np.all(got == got[0])
        near(got[:1], ref, f"{method} n_f={n_f} n_t={n_t} copies={c}", k2)
        assert pk["index"][0] == rk["index"][0] or \
            ref[0, pk["index"][0]] >= rk["power"][0] * (1 - 1e-9)


@pytest.mark.parametrize("n_t", [2, 3, 4, 5, 6])
def test_few_points(dev, n_t):
    rng = np.random.default_rng(70 + n_t)
    series = [(np.sort(rng.uniform(0, 50, n_t)), rng.normal(size=n_t)) for _ in range(6)]
    off, t, y = synth.pack(series)
    ora, _ = oracle.batch(off, t, y, 0.05, 5.0, 3000)
    got, _ = call(dev, off, t, y, None, 0.05, 5.0, 3000, 0, "standard")
    ref, _ = call(dev, off, t, y, None, 0.05, 5.0, 3000, 2, "standard")
    # near a vanishing denominator any FP64 evaluation loses eps kappa^2
    k2 = np.stack([shifted_condition(a, 0.05, 5.0, 3000) for a, _ in series])
    near(got, ora, f"oracle n_t={n_t}", k2)
    near(got, ref, f"plain n_t={n_t}", k2)


def shifted_condition(t, lo, hi, n_f):
    f = lo + (hi - lo) / n_f * np.arange(n_f)
    r = np.abs(np.exp(4j * np.pi * np.outer(f, t - t.mean())).sum(axis=1))
    return (len(t) + r) / np.maximum(len(t) - r, 1e-300 + 1e-12 * len(t))


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("stretch", [1.0, 1e3, 1e6, 1e9])
def test_spans(dev, method, stretch):
    """Spans up to 1e9 times ten years: the grid's rounding reaches the phases
    through the residual sums, and beyond their range bin by bin."""
    t, y, _ = synth.sine_object(120, 8)
    dy = np.random.default_rng(4).uniform(0.03, 0.08, 120)
    off = np.array([0, 120, 240], dtype=np.int64)
    args = (dev, off, np.tile(t * stretch, 2), np.tile(y, 2), np.tile(dy, 2), 0.5, 24.0, 1500)
    got, _ = call(*args, 0, method)
    ref, _ = call(*args, 2, method)
    near(got, ref, f"{method} x{stretch:g}")


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("unit", [lsp.CYCLES, lsp.ANGULAR])
@pytest.mark.parametrize("normalize", [True, False])
@pytest.mark.parametrize("order", [lsp.ORDER_INPUT, lsp.ORDER_LPT])
def test_equals_plain_kernel(dev, method, unit, normalize, order):
    """Objects of every status, times in no order, integer days (bins where a
    regressor vanishes) and f = 0, magnitudes of any scale."""
    rng = np.random.default_rng(21)
    series = []
    for n, scale in ((300, 1.0), (40, 1e-30), (90, 1e20), (17, 1.0)):
        t, y, _ = synth.sine_object(n, int(rng.integers(1 << 30)))
        p = rng.permutation(n)
        series.append((t[p], y[p] * scale))
    t, y, _ = synth.sine_object(50, 3)
    series += [(np.arange(64.0), rng.normal(size=64)), (t, np.full(50, 2.0)),
               (t, np.where(np.arange(50) == 7, np.nan, y)), (np.zeros(0), np.zeros(0)),
               (t[:1], y[:1])]
    off, t, y = synth.pack(series)
    dy = rng.uniform(0.03, 0.08, len(t))
    args = (dev, off, t, y, dy, 0.0, 2.0, 3001)
    got, gk = call(*args, 0, method, unit=unit, normalize=normalize, order=order)
    ref, rk = call(*args, 2, method, unit=unit, normalize=normalize, order=order)
    top = np.nanmax(np.where(np.isnan(ref), 0.0, ref), axis=1, keepdims=True)
    top = np.where(top > 0.0, top, 1.0)  # on the scale of each row's largest power
    k2 = np.zeros_like(ref)
    if method == "generalized":
        f = 2.0 / 3001 * np.arange(3001) / (2 * np.pi if unit == lsp.ANGULAR else 1.0)
        for o in range(5):
            k2[o] = np.minimum(moment_condition(t[off[o]:off[o + 1]], dy[off[o]:off[o + 1]], f), 1e12)
    near(got / top, ref / top, method, k2)
    assert np.array_equal(gk["status"], rk["status"])
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    for o in np.nonzero(rk["status"] == lsp.OBJ_OK)[0]:
        assert gk["power"][o] == got[o, gk["index"][o]] == got[o].max()
