"""The matrix-core sums of the FP32 form (every tuning field left to the
library) against the oracle and against the vector kernels (needs an MI355X).

Tolerance.  Each factor's phase carries at most one FP32 rounding of a reduced
phase (2^-25 cycles, 1.9e-7 rad) and the hardware sine or cosine of it, and its
split into two f16 halves drops at most 2^-24: with both factors of a product
an observation's term is off by less than 1e-6 of its magnitude.  The
normalised power is a squared projection, so it moves by at most twice that
times sqrt(P) <= 1, divided by the smaller shifted denominator's fraction of
N, which is above 1/32 wherever the FP64 fix-up does not recompute the bin:
|dP| <= 2 * 1e-6 * 32 = 6.4e-5.  The vector kernels meet the same bound, so
the two differ by at most twice that.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402
from test_gpu_parity import cuda, dev, oracle, run_batch, run_single, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu

ATOL = 2 * 1e-6 * 32


def close(got, ref, what, atol=ATOL):
    both_nan = np.isnan(got) & np.isnan(ref)
    err = np.where(both_nan, 0.0, np.abs(got - ref))
    say(f"    {what}: max |dP| {err.max():.3g}")
    assert np.all(err <= atol), what


def peak_near(row, i, atol=ATOL):
    return row[i] >= row.max() - 2 * atol


# Below one block of 64 bins, around it, around a wave's 2,048 bins and a
# workgroup's 8,192
@pytest.mark.parametrize("n_f", [1, 31, 64, 65, 2047, 2048, 2049, 4097, 8192, 8193, 20000])
def test_bin_edges(dev, n_f):
    w = synth.make_workload("batch_10k", n_obj=5)
    ora_pg, _ = oracle.batch(w.offsets, w.t, w.y, w.f_min, w.f_max, n_f)
    pg, pk = run_batch(dev, w.offsets, w.t, w.y, w.f_min, w.f_max, n_f, form=lsp.FORM_FP32P)
    close(pg, ora_pg, f"batch n_f={n_f}")
    assert all(peak_near(ora_pg[o], pk["index"][o]) for o in range(w.n_obj))
    t, y = w.obj(2)
    pg, pk = run_single(dev, t, y, w.f_min, w.f_max, n_f, form=lsp.FORM_FP32P)
    close(pg, ora_pg[2], f"single n_f={n_f}")
    assert peak_near(ora_pg[2], pk["index"])


# Around the 16 observations of a matrix instruction, a workgroup's round of
# slices, and one staging pass of the batch (256) and of a single series (1,024)
@pytest.mark.parametrize("n_t", [2, 3, 15, 16, 17, 64, 65, 129, 255, 256, 257, 1023, 1025, 2100])
def test_observation_edges(dev, n_t):
    t, y, _ = synth.sine_object(n_t, 1000 + n_t)
    n_f = 3000
    ora_pg, _ = oracle.single(t, y, 1.0, 12.0, n_f)
    pg, _ = run_single(dev, t, y, 1.0, 12.0, n_f, form=lsp.FORM_FP32P)
    close(pg, ora_pg, f"single n_t={n_t}")
    off, tt, yy = synth.pack([(t, y), (t[: n_t // 2], y[: n_t // 2]), (t, -y)])
    pg, pk = run_batch(dev, off, tt, yy, 1.0, 12.0, n_f, form=lsp.FORM_FP32P)
    close(pg[0], ora_pg, f"batch n_t={n_t}")
    close(pg[2], ora_pg, f"batch n_t={n_t}, negated")
    assert pk["status"][0] == lsp.OBJ_OK


@pytest.mark.parametrize("scale", [1e-30, 1e-6, 1.0, 3e4, 1e15])
def test_magnitude_ranges(dev, scale):
    """Magnitudes of any scale, and one outlier 1e3 times the rest."""
    t, y, _ = synth.sine_object(400, 5)
    out = y.copy()
    out[123] = 300.0
    series = [(t, y * scale), (t, out * scale), (t, (y + 1e3) * scale)]
    off, tt, yy = synth.pack(series)
    ora_pg, _ = oracle.batch(off, tt, yy, 1.0, 12.0, 2500)
    pg, _ = run_batch(dev, off, tt, yy, 1.0, 12.0, 2500, form=lsp.FORM_FP32P)
    close(pg, ora_pg, f"scale {scale}")
    pg, _ = run_single(dev, t, out * scale, 1.0, 12.0, 2500, form=lsp.FORM_FP32P)
    close(pg, ora_pg[1], f"single, scale {scale}")


def _mixed(seed):
    """Objects of every status among ordinary ones, times in no order."""
    rng = np.random.default_rng(seed)
    series = []
    for n in (300, 40, 17, 700, 90, 33, 260):
        t, y, _ = synth.sine_object(n, int(rng.integers(1 << 30)))
        p = rng.permutation(n)
        series.append((t[p], y[p]))
    t, y, _ = synth.sine_object(50, 3)
    bad = np.where(np.arange(50) == 7, np.nan, y)
    return series + [(t, np.full(50, 2.0)), (t, bad), (np.zeros(0), np.zeros(0)),
                     (t[:1], y[:1]), (np.arange(64.0), rng.normal(size=64))]


@pytest.mark.parametrize("unit", [lsp.CYCLES, lsp.ANGULAR])
@pytest.mark.parametrize("normalize", [True, False])
@pytest.mark.parametrize("subtract_mean", [True, False])
@pytest.mark.parametrize("pgram_dtype", [lsp.PGRAM_F32, lsp.PGRAM_F64])
@pytest.mark.parametrize("order", [lsp.ORDER_INPUT, lsp.ORDER_LPT])
def test_equals_vector_kernels(dev, unit, normalize, subtract_mean, pgram_dtype, order):
    """Every option the matrix path accepts, against the vector kernels (an
    explicit k_per_lane): powers, statuses, fill values and peaks; the grid
    starts at f = 0, where the FP64 fix-up takes over on both sides."""
    off, t, y = synth.pack(_mixed(11))
    kw = dict(form=lsp.FORM_FP32P, unit=unit, normalize=normalize, subtract_mean=subtract_mean,
              pgram_dtype=pgram_dtype, order=order)
    args = (dev, off, t, y, 0.0, 6.0, 5003)
    pg, pk = run_batch(*args, **kw)
    ref, rk = run_batch(*args, k=16, **kw)
    top = np.nanmax(ref, axis=1, keepdims=True)  # unnormalised power: on the scale of 1
    top = np.where(np.isfinite(top) & (top > 1.0), top, 1.0)
    close(pg / top, ref / top, "matrix against vector", 2 * ATOL)
    assert np.array_equal(np.isnan(pg), np.isnan(ref))
    assert np.array_equal(pk["status"], rk["status"])
    for o in np.nonzero(rk["status"] == lsp.OBJ_OK)[0]:
        assert peak_near(ref[o] / top[o], pk["index"][o], 2 * ATOL)
        assert np.float32(pk["power"][o]) == np.float32(pg[o, pk["index"][o]])
    assert np.all(pk["index"][rk["status"] != lsp.OBJ_OK] == -1)
    _, only = run_batch(*args, pgram=False, **kw)
    assert only.tobytes() == pk.tobytes()


def test_rows_equal_whole_grid(dev):
    """Bands of any width give the bins' whole-grid powers: the matrix path's
    blocks start at the band, so they are equal within the bound."""
    w = synth.make_workload("batch_10k", n_obj=9)
    n_f = 20000
    ref, _ = run_batch(dev, w.offsets, w.t, w.y, w.f_min, w.f_max, n_f, form=lsp.FORM_FP32P)
    for band in (40, 2000, 2100, 5000, 9000):
        n_b = -(-n_f // band)
        rows = np.tile(np.arange(n_b, dtype=np.int32), w.n_obj)
        pg = torch.full((w.n_obj, n_f), -7.0, dtype=torch.float32, device=dev)
        r = lsp.Rows(cuda(w.offsets, dev, torch.int64), cuda(w.t, dev), cuda(w.y, dev), w.f_min,
                     w.f_max, n_f, None, cuda(rows, dev, torch.int32), band, n_b, pgram=pg)
        r()
        torch.cuda.synchronize()
        got = pg.double().cpu().numpy()
        close(got, ref, f"bands of {band}", 2 * ATOL)
        pk = r.peaks()
        assert all(pk["power"][o] == got[o, pk["index"][o]] == got[o].max()
                   for o in range(w.n_obj))


# ---- generalized form: 1,024-bin wave tiles, 32 observations an instruction

@pytest.mark.parametrize("n_f", [1, 33, 64, 1023, 1025, 4096, 4097, 9000])
@pytest.mark.parametrize("n_t", [4, 31, 33, 64, 255, 257, 1030])
def test_generalized_edges(dev, n_f, n_t):
    """Around the tile sizes, against the vector kernels (an explicit
    k_per_lane), on an ordinary series and one with errors over four decades;
    both are within the bound of the oracle, so within twice it of each other."""
    rng = np.random.default_rng(n_t)
    t, y, _ = synth.sine_object(n_t, 2000 + n_t)
    dy = np.concatenate([rng.uniform(0.03, 0.08, n_t), 10.0 ** rng.uniform(-4.0, 0.0, n_t)])
    off, tt, yy = synth.pack([(t, y), (t, -y)])
    kw = dict(form=lsp.FORM_FP32P, method="generalized", pgram_dtype=lsp.PGRAM_F64)
    got, ref = (lsp.Periodogram(cuda(tt, dev), cuda(yy, dev), 1.0, 12.0, n_f,
                                offsets=cuda(off, dev, torch.int64), dy=cuda(dy, dev), k=k, **kw)()
                for k in (0, 16))
    close(got.pgram.cpu().numpy(), ref.pgram.cpu().numpy(), f"n_f={n_f} n_t={n_t}", 2 * ATOL)
    pk, rk = got.peaks(), ref.peaks()
    assert np.array_equal(pk["status"], rk["status"])
    one = lsp.Periodogram(cuda(t, dev), cuda(y, dev), 1.0, 12.0, n_f, dy=cuda(dy[:n_t], dev),
                          **kw)()
    close(one.pgram.cpu().numpy(), ref.pgram.cpu().numpy()[:1], "single", 2 * ATOL)
    row = ref.pgram.cpu().numpy()[0]
    assert peak_near(row, pk["index"][0], 2 * ATOL)
    assert peak_near(row, one.peaks()["index"][0], 2 * ATOL)
