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
