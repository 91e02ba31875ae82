"""The residual of the grid's rounding in the FP64 matrix-core form, against the
plain FP64 kernel (an explicit k_per_lane) (needs an MI355X).

Tolerance.  A term of a sum is off by less than 8 * 2^-53 = 9e-16 of its size (the
rounded sines and cosines of two factors, three products, the sums); the errors
of n terms add as their root, as the terms themselves do in most bins, so a sum
is off by about that fraction of its size, the power by twice, and the two forms
by four times, 4e-15, of each other.  The norm of the difference over a grid is
held to 1e-14 of the powers' norm.  With the residual's sums in single f16
values it is 3e-14 at 300 cycles a day on ten years, without the residual 1e-10.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402,F401
from test_gpu_fx import call  # noqa: E402
from test_gpu_parity import dev, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("f_max", [24.0, 300.0])
@pytest.mark.parametrize("n_t", [60, 1000])
@pytest.mark.parametrize("copies", [1, 40])  # the shared tile, a tile a wave
def test_as_accurate_as_term_by_term(dev, method, f_max, n_t, copies):
    t, y, _ = synth.sine_object(n_t, 600 + n_t)
    dy = np.random.default_rng(n_t).uniform(0.03, 0.08, n_t)
    n_f = 10_000
    off = np.arange(copies + 1, dtype=np.int64) * n_t
    args = [np.tile(v, copies) for v in (t, y, dy)]
    got, _ = call(dev, off, *args, 0.5, f_max, n_f, 0, method)
    ref, _ = call(dev, None, t, y, dy, 0.5, f_max, n_f, 2, method)
    err = np.linalg.norm(got - ref, axis=1).max() / np.linalg.norm(ref)
    say(f"    {method} f_max={f_max:g} n_t={n_t} x{copies}: {err:.3g}")
    assert err <= 1e-14
