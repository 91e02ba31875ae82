"""Which kernels a call takes, as far as the host shows it (no GPU)."""
import pytest

from paper_2105_04006_amd import lsp

SHAPES = [(1, 100), (1, 20_000), (3, 64), (20, 300), (48, 40_000), (2000, 16), (2000, 130),
          (2000, 257), (2000, 512), (2000, 2049), (30_000, 9000)]


@pytest.mark.parametrize("gen", [False, True])
def test_fp64_workspace_does_not_depend_on_the_observations(gen):
    """A program sizes its workspace for the most observations it expects: the
    route may depend on their number, the bytes may not."""
    opt = lsp.make_options(form=lsp.FORM_FP64, order=lsp.ORDER_INPUT)
    for n_obj, n_f in SHAPES:
        g = lsp.make_grid(0.5, 24.0, n_f)
        need = {lsp.gen_workspace_bytes(n_obj, n_obj * n, g, opt) if gen else
                lsp.workspace_bytes(n_obj, n_obj * n, g, opt)
                for n in (0, 1, 3, 5, 20, 30, 90, 150, 250, 1000, 100_000)}
        assert len(need) == 1 and need.pop() > 0, (n_obj, n_f)


def test_launch_names_the_kernels_that_run():
    """The described launch says which kernels the call runs and, for the
    matrix-core ones, their shape; the resolved options give the same launch."""
    f32, f64 = lsp.FORM_FP32P, lsp.FORM_FP64
    cases = [  # n_obj, n_obs, n_f, options, generalized, expected matrix shape
        (1, 256, 10_000, dict(form=f32), False, (2048, 5, 8, 1, 1)),
        (1, 4096, 500_000, dict(form=f32), False, (2048, 245, 8, 1, 1)),
        (1, 20_000, 10_000, dict(form=f32), False, (2048, 195, 8, 1, 39)),
        (1, 20_000, 10_000, dict(form=f32), True, (1024, 250, 8, 1, 25)),
        (2500, 650_000, 250_000, dict(form=f32), False, (2048, 2500 * 31, 4, 0, 1)),
        (300, 50_000, 100_003, dict(form=f32), True, (1024, 300 * 25, 4, 0, 1)),
        (48, 24_000, 40_000, dict(form=f64), False, (512, 48 * 20, 4, 0, 1)),
        (1, 256, 10_000, dict(form=f64), False, (512, 20, 8, 1, 1)),
        (2000, 200_000, 64, dict(form=f64), False, None),   # a small grid
        (2000, 6000, 10_000, dict(form=f64), False, None),  # three points an object
        (1, 256, 10_000, dict(form=f32, k=16), False, None),
        (1, 256, 10_000, dict(form=f32, kernels=lsp.KERNELS_VECTOR), False, None),
        (1, 256, 10_000, dict(form=f32, k=16, waves=4, kernels=lsp.KERNELS_MATRIX), False,
         (2048, 5, 8, 1, 1)),
    ]
    for n_obj, n_obs, n_f, kw, gen, shape in cases:
        g = lsp.make_grid(0.5, 24.0, n_f)
        opt = lsp.make_options(**kw)
        d = lsp.describe_launch(n_obj, n_obs, g, opt, gen)
        assert d["kernels"] == (lsp.KERNELS_MATRIX if shape else lsp.KERNELS_VECTOR), d
        got = d["matrix"] and tuple(d["matrix"][k] for k in ("wave_bins", "n_items", "waves",
                                                             "shared", "parts"))
        assert got == shape, (n_obj, n_f, kw, d["matrix"])
        again = lsp.Options()
        for name, _ in lsp.Options._fields_:
            setattr(again, name, d[name])
        d2 = lsp.describe_launch(n_obj, n_obs, g, again, gen)
        assert (d2["kernels"], d2["matrix"]) == (d["kernels"], d["matrix"])


def test_kernels_field_takes_the_reserved_one():
    """Unknown values of the field that used to be reserved are ignored, as before."""
    g = lsp.make_grid(0.5, 24.0, 10_000)
    opt = lsp.make_options(form=lsp.FORM_FP32P)
    want = lsp.describe_launch(1, 256, g, opt)
    for v in (-1, 3, 77):
        opt.kernels = v
        assert lsp.describe_launch(1, 256, g, opt) == want


@pytest.mark.parametrize("form", [lsp.FORM_FP32P, lsp.FORM_FP64])
def test_generalized_workspace_serves_the_standard_form(form):
    """A program may size one buffer for both methods from the generalized call."""
    opt = lsp.make_options(form=form)
    for n_obj in (1, 2, 40, 3000):
        for n_f in (1, 500, 2000, 10_000, 60_000, 130_000, 500_000, 3_000_000):
            for n in (1, 30, 600, 1500, 5000, 20_000, 1_000_000):
                g = lsp.make_grid(0.5, 24.0, n_f)
                std = lsp.workspace_bytes(n_obj, n_obj * n, g, opt)
                assert 0 < std <= lsp.gen_workspace_bytes(n_obj, n_obj * n, g, opt), (n_obj, n_f, n)
