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


# one level: output edges that leave boxes of voxels partly empty (26, 19, 5), and full ones (32, 16, 8)
@pytest.mark.parametrize("edge", [26, 19, 5, 32, 16, 8])
def test_weight_gradient_of_infinite_input(edge):
    """A voxel in the last corner meets tap 0 of an axis only at an output that does not exist."""
    net = L.WarmStartNet(channels=(5,), in_size=edge, seed=4)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(2, 2, edge, edge, edge, device="cuda", generator=g)
    dout = torch.randn(2, 3, edge, edge, edge, device="cuda", generator=g)
    grads = []
    for value in (0.0, float("inf")):
        x[1, 1, -1, -1, -1] = value
        net.forward(x)
        net.zero_grad()
        net.backward(dout)
        grads.append(torch.from_numpy(net.get(1)[:5 * 2 * 27]).reshape(5, 2, 3, 3, 3))
    met = torch.zeros(2, 3, 3, 3, dtype=torch.bool)
    met[1, 1:, 1:, 1:] = True
    assert not torch.isfinite(grads[1][:, met]).all()
    assert torch.isfinite(grads[1][:, ~met]).all()
