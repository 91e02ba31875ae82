"""Bins of the FP64 matrix-core form whose sums are taken term by term: listed
ones (a vanishing denominator), all of an object's past the residual's range, and
all of an object of a few points; against the plain FP64 kernel (an explicit
k_per_lane) (needs an MI355X).

Near a vanishing denominator an FP64 evaluation of the standard form loses eps
kappa^2 of the power, kappa the condition of the bin's moment matrix; elsewhere
both hold the FP64 form's bound, |dP| <= 1e-9 max(P, 1e-3).  The generalized
form's moments lose more, in the subtraction of the weighted means (the plain
kernel is off by 1e-5 where a regressor's variance is 1e-12), so there both are
compared with an extended-precision evaluation: they add the same terms in
another order, so their errors have the same law, and the norm over the bins,
which a few of the worst make up, may differ by a factor of 8.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402
from test_gpu_fx import call, near, shifted_condition  # noqa: E402
from test_gpu_parity import dev, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu


def exact_generalized(t, y, dy, f):
    """Generalized power in extended precision, and the smaller variance of the
    regressors as a fraction of the total weight."""
    ld = np.longdouble
    w = 1 / dy.astype(ld) ** 2
    w /= w.sum()
    yc = y - (w * y).sum()
    turn = np.multiply.outer(f.astype(ld), t.astype(ld) - ld(t[0]))
    ph = 8 * np.arctan(ld(1)) * (turn - np.rint(turn))
    c, s = np.cos(ph), np.sin(ph)
    c -= (c @ w)[:, None]
    s -= (s @ w)[:, None]
    cc, ss, cs, yx, ys = (c * c) @ w, (s * s) @ w, (c * s) @ w, c @ (w * yc), s @ (w * yc)
    least = 0.5 * (cc + ss - np.sqrt((cc - ss) ** 2 + 4 * cs * cs))
    with np.errstate(divide="ignore", invalid="ignore"):
        p = (yx * yx * ss + ys * ys * cc - 2 * yx * ys * cs) / (cc * ss - cs * cs)
    return p / (w * yc * yc).sum(), least


def check(dev, method, series, lo, hi, n_f, what):
    rng = np.random.default_rng(5)
    off, t, y = synth.pack(series)
    dy = rng.uniform(0.03, 0.08, len(t))
    got, gk = call(dev, off, t, y, dy, lo, hi, n_f, 0, method)
    ref, _ = call(dev, off, t, y, dy, lo, hi, n_f, 2, method)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    for o in range(len(series)):
        assert gk["power"][o] == got[o, gk["index"][o]] == got[o].max()
    if method == "standard":
        times = {id(a): a for a, _ in series}  # (copies share theirs)
        k2 = {i: np.minimum(shifted_condition(a, lo, hi, n_f) ** 2, 1e12) for i, a in times.items()}
        k2 = np.stack([k2[id(a)] for a, _ in series])
        near(got, ref, what, k2)
        return
    f = lo + (hi - lo) / n_f * np.arange(n_f)
    for o in range(0, len(series), max(1, len(series) // 3)):
        own = slice(off[o], off[o + 1])
        p, least = exact_generalized(t[own], y[own], dy[own], f)
        sure = least > 4e-12  # well above the denominators that are dropped (1e-12)
        assert np.all(np.abs(got[o] - ref[o])[least > 1e-3] <= 2e-12)
        e_got, e_ref, top = (np.linalg.norm(v[sure].astype(float))
                             for v in (got[o] - p, ref[o] - p, p))
        say(f"    {what}: object {o}, error {e_got:.3g}, plain kernel {e_ref:.3g} of {top:.3g}")
        assert e_got <= 8.0 * e_ref + 1e-14 * top


# A list of a few bins, of some dozens and of all of a workgroup's; one staging
# pass and several; the shared tile (2 objects) and a tile a wave (200 objects)
@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n_t", [30, 256, 300])
@pytest.mark.parametrize("copies", [2, 200])
@pytest.mark.parametrize("kind", ["days", "clumps", "night"])
def test_listed_bins(dev, method, n_t, copies, kind):
    rng = np.random.default_rng(n_t)
    if kind == "days":       # integer days: f = 0, 1/2, 1, ...
        t = np.sort(rng.choice(4000, n_t, replace=False)).astype(np.float64)
        lo, hi = 0.0, 2.0
    elif kind == "clumps":   # two nights a year apart
        t = np.sort(np.where(np.arange(n_t) % 2, 365.0, 0.0) + 0.02 * rng.random(n_t))
        lo, hi = 0.5, 12.0
    else:                    # one hour, periods of days
        t = np.sort(0.04 * rng.random(n_t))
        lo, hi = 0.0, 0.3
    y = rng.normal(size=n_t)
    check(dev, method, [(t, y if c % 2 else -y) for c in range(copies)], lo, hi, 3001,
          f"{method} {kind} n_t={n_t} x{copies}")


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n_t", [7, 256, 601])
@pytest.mark.parametrize("n_f,copies", [(1, 1), (511, 1), (2049, 1), (2049, 200), (6000, 60)])
def test_past_the_residuals_range(dev, method, n_t, n_f, copies):
    """500 cycles a day on ten years."""
    t, y, _ = synth.sine_object(n_t, 40 + n_t)
    check(dev, method, [(t, (1.0 + c) * y) for c in range(copies)], 400.0, 500.0, n_f,
          f"{method} n_t={n_t} n_f={n_f} x{copies}")


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n_t", [4, 5, 6, 7])
@pytest.mark.parametrize("copies", [3, 300])
def test_few_points_batches(dev, method, n_t, copies):
    rng = np.random.default_rng(90 + n_t)
    series = [(np.sort(rng.uniform(0, 50, n_t)), rng.normal(size=n_t)) for _ in range(copies)]
    check(dev, method, series, 0.05, 5.0, 3000, f"{method} n_t={n_t} x{copies}")
