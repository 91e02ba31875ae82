"""Features of objects whose seasons differ in magnitude by many decades, against
the FP64 feature reference (needs an MI355X).

A group's spectrum is normalised by the group's own squares, so a season far
below the object's largest magnitudes counts as much as any other.  The power of
a group is held to the FP32 form's bound (test_gpu_mx.py), and so is the mean
over the groups."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import features_ref  # noqa: E402
from paper_2105_04006_amd import synth  # noqa: E402
from test_gpu_features import assert_features_close, gpu_features  # noqa: E402
from test_gpu_mx import ATOL  # noqa: E402
from test_gpu_parity import dev  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ratio", [1.0, 1e-4, 1e-7, 1e-9])
def test_seasons_of_different_magnitudes(dev, ratio):
    rng = np.random.default_rng(17)

    def season(n, start, scale):
        t = start + np.sort(rng.uniform(0, 50, n))
        y = np.sin(2 * np.pi * 3.3 * t) + 0.3 * rng.normal(size=n)
        return t, scale * (y - y.mean())  # (the object's mean stays near zero)

    series = []
    for sizes in ((40, 60, 30), (20, 300, 290), (9, 4, 8, 17), (500, 33)):
        for order in (1, -1):
            scales = [1.0, ratio, ratio ** 0.5, ratio][:len(sizes)][::order]
            parts = [season(n, 200.0 * i, s) for i, (n, s) in enumerate(zip(sizes, scales))]
            series.append(tuple(np.concatenate(v) for v in zip(*parts)))
    off, t, y = synth.pack(series)
    ref = features_ref.features(off, t, y, 1.0, 12.0)
    got = gpu_features(dev, off, t, y, 1.0, 12.0)
    assert_features_close(got, ref, f"ratio {ratio:g}", coarse_atol=ATOL)
