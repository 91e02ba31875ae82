"""The `kernels` option: a call described and repeated with its resolved options,
and each kind of kernels asked for by name (needs an MI355X)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_04006_amd import lsp, synth  # noqa: E402
from test_gpu_parity import cuda, dev  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["standard", "generalized"])
@pytest.mark.parametrize("form,k", [(lsp.FORM_FP32P, 16), (lsp.FORM_FP64, 2)])
def test_kernels_by_name(dev, method, form, k):
    w = synth.make_workload("batch_10k", n_obj=6)
    dy = np.random.default_rng(1).uniform(0.03, 0.08, len(w.t))

    def call(**kw):
        p = lsp.Periodogram(cuda(w.t, dev), cuda(w.y, dev), w.f_min, w.f_max, 5003,
                            offsets=cuda(w.offsets, dev, torch.int64), form=form, method=method,
                            dy=cuda(dy, dev) if method == "generalized" else None,
                            pgram_dtype=lsp.PGRAM_F64, **kw)()
        torch.cuda.synchronize()
        return p, p.pgram.cpu().numpy()

    plain, matrix = call()
    tuned, vector = call(k=k)
    assert plain.launch()["matrix"] and not tuned.launch()["matrix"]
    assert not np.array_equal(matrix, vector)
    assert np.array_equal(call(k=k, kernels=lsp.KERNELS_MATRIX)[1], matrix)
    assert np.array_equal(call(k=k, kernels=lsp.KERNELS_VECTOR)[1], vector)
    for p, got in ((plain, matrix), (tuned, vector)):
        d = p.launch()
        same = call(k=d["k_per_lane"], waves=d["waves_per_wg"], t_split=d["t_split"],
                    schedule=d["schedule"], recurrence=d["recurrence"],
                    wave_split=d["wave_split"], obs_read=d["obs_read"],
                    seed_trig=d["seed_trig"], order=d["order"], kernels=d["kernels"])[1]
        assert np.array_equal(same, got)
