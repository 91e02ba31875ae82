"""Peaks written by the last workgroup of the kernel before, and by a kernel of
their own: around the number of objects and of workgroups at which one takes
over from the other (needs an MI355X).

The peak of a call is exactly the first maximal bin of the periodogram that the
same call stores, so no tolerance is needed; calls repeat on one plan, eagerly
and as a graph, on changed data, so that a counter left over would show."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [  # (objects, observations, bins, form): 0 objects is a single series
    (1, 70, 3000, lsp.FORM_FP32P), (255, 24, 1500, lsp.FORM_FP32P),
    (256, 24, 1500, lsp.FORM_FP32P), (257, 24, 1500, lsp.FORM_FP32P),
    (200, 24, 330 * 1024, lsp.FORM_FP32P),   # tiles around 256 x 256
    (0, 70, 5000, lsp.FORM_FP32P), (0, 300, 256 * 1024, lsp.FORM_FP32P),
    (0, 300, 256 * 1024 + 1, lsp.FORM_FP32P),
    (0, 70, 300, lsp.FORM_FP64), (0, 300, 256 * 512, lsp.FORM_FP64),
    (0, 300, 256 * 512 + 1, lsp.FORM_FP64), (1, 300, 5000, lsp.FORM_FP64),
    (2, 300, 5000, lsp.FORM_FP64),
]


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("n_obj,n,n_f,form", CASES)
def test_peaks_are_the_stored_maxima(n_obj, n, n_f, form, method):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n_obj + n_f)
    k = max(n_obj, 1)
    t = torch.rand(k * n, dtype=torch.float64, device="cuda:0", generator=gen) * 1000.0
    y = torch.randn(k * n, dtype=torch.float64, device="cuda:0", generator=gen)
    off = torch.arange(k + 1, device="cuda:0") * n if n_obj else None
    dt = lsp.PGRAM_F32 if form == lsp.FORM_FP32P else lsp.PGRAM_F64
    # from f = 0: the first bins are ill-conditioned (the fix-up's)
    p = lsp.Periodogram(t, y, 0.0, 4.0, n_f, offsets=off, form=form, method=method,
                        pgram_dtype=dt)

    def check(what):
        torch.cuda.synchronize()
        print(f"peaks {n_obj} x {n} x {n_f} {method} {what}", flush=True)
        pg = torch.nan_to_num(p.pgram.reshape(k, n_f), nan=-1.0)
        pk = p.peaks()
        first = torch.argmax(pg, dim=1).cpu().numpy()
        top = pg.max(dim=1).values.cpu().numpy().astype(np.float64)
        at = pg.cpu().numpy()[np.arange(k), pk["index"]].astype(np.float64)
        assert np.array_equal(at, top) and np.array_equal(pk["power"], top)
        assert np.all(pk["index"] <= first)
        p.peaks_raw.zero_()

    for rep in range(2):
        p()
        check(f"call {rep}")
        y.neg_().add_(torch.randn(k * n, dtype=torch.float64, device="cuda:0", generator=gen))
    plan = p.capture()
    for rep in range(3):
        plan()
        check(f"replay {rep}")
        y.neg_().add_(torch.randn(k * n, dtype=torch.float64, device="cuda:0", generator=gen))
