"""FP64 calls on either side of the lines between the vector kernel and the
matrix-core kernels (bins of a row, mean points per object), against an explicit
vector shape (k_per_lane), with the FP64 form's bound (needs an MI355X)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402
from test_gpu_fx import call, near  # noqa: E402
from test_gpu_parity import cuda, dev  # noqa: E402,F401

pytestmark = pytest.mark.gpu


def batch(n_obj, points):
    """Pairs of objects with `points` points on average, from 24 on."""
    rng = np.random.default_rng(points)
    apart = rng.integers(0, points - 24 + 1, n_obj // 2)
    n = np.stack([points - apart, points + apart], axis=1).ravel()
    assert len(n) == n_obj and n.sum() == points * n_obj
    series = [synth.sine_object(int(m), 50 + i % 20)[:2] for i, m in enumerate(n)]
    off, t, y = synth.pack(series)
    return off, t, y, rng.uniform(0.03, 0.08, len(t))


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n_f,points", [(16, 60), (128, 60), (129, 99), (129, 100), (129, 101),
                                        (256, 200), (256, 201), (257, 32), (512, 32), (512, 33)])
def test_lines(dev, method, n_f, points):
    off, t, y, dy = batch(530, points)
    got, gk = call(dev, off, t, y, dy, 1.0, 12.0, n_f, 0, method)
    ref, rk = call(dev, off, t, y, dy, 1.0, 12.0, n_f, 2, method)
    near(got, ref, f"{method} n_f={n_f} points={points}", 1e4)
    assert np.array_equal(gk["status"], rk["status"])
    assert np.all(gk["power"] == got.max(axis=1))


@pytest.mark.parametrize("band", [100, 128, 256, 300, 512, 700])
def test_bands(dev, band):
    off, t, y, _ = batch(530, 60)
    n_f, per = 8 * band - 5, 2
    rows = np.random.default_rng(band).integers(0, 8, 530 * per).astype(np.int32)
    pg = torch.full((530, n_f), -7.0, dtype=torch.float64, device=dev)
    r = lsp.Rows(cuda(off, dev, torch.int64), cuda(t, dev), cuda(y, dev), 1.0, 12.0, n_f, None,
                 cuda(rows, dev, torch.int32), band, per, pgram=pg, pgram_dtype=lsp.PGRAM_F64,
                 form=lsp.FORM_FP64)
    r()
    torch.cuda.synchronize()
    got = pg.cpu().numpy()
    ref, _ = call(dev, off, t, y, None, 1.0, 12.0, n_f, 2, "standard")
    pk = r.peaks()
    for o in range(530):
        inside = np.zeros(n_f, bool)
        for b in rows[per * o:per * o + per]:
            inside[b * band:(b + 1) * band] = True
        assert np.all(got[o, ~inside] == -7.0)
        near(got[o, inside], ref[o, inside], f"band={band} object {o}", 1e4)
        assert pk["power"][o] == got[o, inside].max() == got[o, pk["index"][o]]
