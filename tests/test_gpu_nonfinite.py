"""Infinities and NaN stay with the values that are computed from them: where a tile of a kernel runs past a row, a
plane or a grid, what lies there is not multiplied by zero."""
import pytest
import torch

from paper_2006_06823_amd import lddmm_bl as L

pytestmark = pytest.mark.gpu


# (inner axes that end inside a tile of 32, at its end, and bands of one and two tiles; 2D; an axis above 192)
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("precision", [L.FP32, L.BF16_DFT, L.FP64])
@pytest.mark.parametrize("N,K", [((26, 20, 23), (8, 6, 10)), ((70, 18, 34), (18, 8, 12)), ((32, 64, 32), (8, 10, 6)),
                                 ((21, 101, 53), (6, 34, 12)), ((24, 54, 102), (6, 18, 34)), ((50, 61), (14, 18)),
                                 ((200, 20, 18), (40, 8, 6))])
def test_transforms_keep_fields_apart(N, K, precision, bad):
    ctx = L.Context(L.Problem(N, K, nt=1, precision=precision))
    g = torch.Generator(device="cuda").manual_seed(3)
    for call, shape in ((ctx.project, N), (ctx.include, K)):
        x = torch.randn(3, *shape, device="cuda", generator=g, dtype=ctx.dtype)
        ref = call(x, 3)
        for f in range(3):
            y = x.clone()
            y[f] = bad
            got = call(y, 3)
            assert not torch.isfinite(got[f]).any()
            for o in range(3):
                if o != f:
                    assert torch.equal(got[o], ref[o]), (call.__name__, f, o)
