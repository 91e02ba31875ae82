"""The matrix-core kernels that give each wave a tile of its own (calls of more
than 400 tiles, every tuning field left to the library), bin by bin against the
oracle, and outputs past 2^31 elements (needs an MI355X).

Tolerances.  Bin by bin that of test_gpu_mx.py.  Over all bins: a term of a sum is
off by some 2e-7 of its size (the FP32 rounding of its two phases, 1.1e-7 rad
each in the mean square, the hardware sines, the halves' 2^-24), the errors of n
terms add as their root, as the terms do in most bins, and the power is
quadratic, so the norm of the error is near 4e-7 of the powers' norm; it is held
to 1e-6.  (Without one of the products of halves it is some 2e-4.)
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402
from test_gpu_mx import ATOL, close, peak_near  # noqa: E402
from test_gpu_parity import cuda, dev, oracle, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu

COPIES = 140  # of three objects: 420 rows


def norm_error(got, ref):
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


def three(n_t):
    """Three objects: two of n_t points, one shorter."""
    t, y, _ = synth.sine_object(n_t, 4000 + n_t)
    u, z, _ = synth.sine_object(n_t, 4100 + n_t)
    return [(t, y), (u, z), (t[: 1 + n_t // 2], y[: 1 + n_t // 2])]


def copies(dev, series, dy, lo, hi, n_f, waves, bins, **kw):
    """The rows of the three objects from a batch of their copies, all alike."""
    off, t, y = synth.pack(series * COPIES)
    p = lsp.Periodogram(cuda(t, dev), cuda(y, dev), lo, hi, n_f,
                        offsets=cuda(off, dev, torch.int64), form=lsp.FORM_FP32P,
                        method="standard" if dy is None else "generalized",
                        dy=None if dy is None else cuda(np.tile(dy, COPIES), dev), **kw)()
    m = p.launch()["matrix"]
    assert (m["waves"], m["shared"], m["wave_bins"]) == (waves, 0, bins)
    pg = p.pgram.view(COPIES, 3, n_f)
    assert torch.equal(pg, pg[:1].expand_as(pg))
    pk = p.peaks().reshape(COPIES, 3)
    assert np.all(pk == pk[:1])
    return pg[0].double().cpu().numpy(), pk[0]


# One, two and four waves a workgroup (rows of up to 2,048, 4,096 and more bins),
# around the 16 observations of a matrix instruction, a round of slices and the
# 256 of a staging pass
@pytest.mark.parametrize("n_f,waves,n_t", [
    (1, 1, 70), (65, 1, 70), (2047, 1, 70), (2048, 1, 257), (2049, 2, 70), (4095, 2, 255),
    (4096, 2, 600), (4097, 4, 70), (8191, 4, 70), (8193, 4, 257), (20_000, 4, 70),
    (2048, 1, 15), (2048, 1, 16), (2048, 1, 17), (4096, 2, 31), (4096, 2, 33), (4096, 2, 64),
    (8192, 4, 63), (8192, 4, 65), (8192, 4, 127), (8192, 4, 129), (8192, 4, 256), (8192, 4, 513)])
def test_standard_tiles(dev, n_f, waves, n_t):
    series = three(n_t)
    got, pk = copies(dev, series, None, 1.0, 12.0, n_f, waves, 2048)
    off, t, y = synth.pack(series)
    ref, _ = oracle.batch(off, t, y, 1.0, 12.0, n_f)
    close(got, ref, f"n_f={n_f} n_t={n_t}")
    assert all(peak_near(ref[o], pk["index"][o]) for o in range(3))
    assert all(np.float32(pk["power"][o]) == got[o, pk["index"][o]] == got[o].max()
               for o in range(3))
    if n_t >= 64 and n_f >= 2000:
        err = [norm_error(got[o], ref[o]) for o in range(2)]
        say(f"    n_f={n_f} n_t={n_t}: norm of the error {max(err):.3g}")
        assert max(err) <= 1e-6


@pytest.mark.parametrize("n_f,n_t", [
    (1, 70), (33, 70), (1023, 70), (1025, 257), (4095, 255), (4096, 600), (4097, 70), (9000, 70),
    (4096, 31), (4096, 32), (4096, 33), (4096, 63), (4096, 65), (4096, 256), (4096, 513)])
def test_generalized_tiles(dev, n_f, n_t):
    series = three(n_t)
    off, t, y = synth.pack(series)
    dy = np.random.default_rng(n_t).uniform(0.03, 0.08, len(t))
    got, pk = copies(dev, series, dy, 1.0, 12.0, n_f, 4, 1024)
    ref, _ = oracle.gen_batch(off, t, y, dy, 1.0, 12.0, n_f)
    close(got, ref, f"n_f={n_f} n_t={n_t}")
    assert all(peak_near(ref[o], pk["index"][o]) for o in range(3))
    if n_t >= 64 and n_f >= 2000:
        err = [norm_error(got[o], ref[o]) for o in range(2)]
        say(f"    n_f={n_f} n_t={n_t}: norm of the error {max(err):.3g}")
        assert max(err) <= 1e-6


@pytest.mark.parametrize("n_t", [70, 1000, 5000])
@pytest.mark.parametrize("method", ["standard", "generalized"])
def test_shared_tiles_norm_error(dev, method, n_t):
    """The kernels whose waves share a tile, with the same norm."""
    t, y, _ = synth.sine_object(n_t, 4200 + n_t)
    dy = np.random.default_rng(n_t).uniform(0.03, 0.08, n_t)
    gen = method == "generalized"
    p = lsp.Periodogram(cuda(t, dev), cuda(y, dev), 1.0, 12.0, 9000, form=lsp.FORM_FP32P,
                        method=method, dy=cuda(dy, dev) if gen else None)()
    ref, _ = oracle.gen_single(t, y, dy, 1.0, 12.0, 9000) if gen else \
        oracle.single(t, y, 1.0, 12.0, 9000)
    err = norm_error(p.pgram[0].double().cpu().numpy(), ref)
    say(f"    {method} n_t={n_t}: norm of the error {err:.3g}")
    assert p.launch()["matrix"]["shared"] and err <= 1e-6


@pytest.mark.parametrize("form", [lsp.FORM_FP32P, lsp.FORM_FP64])
def test_rows_past_2_31_elements(dev, form):
    """2,201 objects on 1,000,003 bins: rows from 2,148 on start past 2^31."""
    n_obj, n_f = 2201, 1_000_003
    rng = np.random.default_rng(9)
    series = [synth.sine_object(int(n), i)[:2] for i, n in enumerate(rng.integers(20, 40, 31))]
    off, t, y = synth.pack([series[o % 31] for o in range(n_obj)])
    p = lsp.Periodogram(cuda(t, dev), cuda(y, dev), 1.0, 12.0, n_f,
                        offsets=cuda(off, dev, torch.int64), form=form)()
    assert p.launch()["matrix"]
    pk = p.peaks()
    for o in (2199, 2200):
        assert o * n_f > 2 ** 31
        assert torch.equal(p.pgram[o], p.pgram[o % 31])
        for f in ("index", "freq", "period", "power", "status"):
            assert pk[f][o] == pk[f][o % 31]
        ref, _ = oracle.single(*series[o % 31], 1.0, 12.0, n_f)
        close(p.pgram[o].double().cpu().numpy(), ref, f"object {o}")
        assert peak_near(ref, pk["index"][o])


def test_survey_batch_with_default_options(dev):
    """2,000 objects of the lsst_200k population, every option left to the library
    (longest-first order included): peaks of the FP32 form against the FP64 one."""
    w = synth.make_workload("lsst_200k", n_obj=2000)
    args = (cuda(w.t, dev), cuda(w.y, dev), w.f_min, w.f_max, w.n_f)
    kw = dict(offsets=cuda(w.offsets, dev, torch.int64), pgram=False)
    p32 = lsp.Periodogram(*args, form=lsp.FORM_FP32P, **kw)()
    p64 = lsp.Periodogram(*args, form=lsp.FORM_FP64, **kw)()
    a, b = p32.peaks(), p64.peaks()
    assert p32.launch()["matrix"] and p32.launch()["order"] == lsp.ORDER_LPT
    assert np.array_equal(a["status"], b["status"])
    ok = b["status"] == 0
    near = np.abs(a["index"] - b["index"])[ok] <= 1
    d = np.abs(a["power"] - b["power"])[ok]
    say(f"    peaks within a bin {near.mean():.4f}, max |dP| {d.max():.3g}")
    # the peaks' powers differ by the bound; other bins are near-ties
    assert d.max() <= ATOL and near.mean() >= 0.999
