"""Batches whose samples, and samples times channels, exceed 65535 workgroups in a dimension of a launch."""
import pytest
import torch

from paper_2006_06823_amd import lddmm_bl as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,channels", [(65537, 2), (40000, 2)])
def test_large_batch(B, channels):
    """Outputs bitwise those of small batches; weight gradients their sum up to FP32 accumulation: a sum of n terms of
    random signs errs by about sqrt(n) 2^-24 of its terms' norm, n = 64 B < 2^23, and so does the bias' atomic sum."""
    net = L.WarmStartNet(channels=(channels,), in_size=4, seed=6)
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(B, 2, 4, 4, 4, device="cuda", generator=g)
    dout = torch.randn(B, 3, 4, 4, 4, device="cuda", generator=g)
    out = net.forward(x)
    net.zero_grad()
    net.backward(dout)
    grad = torch.from_numpy(net.get(1)).double()
    total = torch.zeros_like(grad)
    squares = torch.zeros_like(grad)
    for lo in range(0, B, 4096):
        part = net.forward(x[lo:lo + 4096].contiguous())
        assert torch.equal(part, out[lo:lo + 4096])
        net.zero_grad()
        net.backward(dout[lo:lo + 4096].contiguous())
        p = torch.from_numpy(net.get(1)).double()
        total += p
        squares += p * p
    assert ((grad - total).abs() <= (64 * B) ** 0.5 * 2.0 ** -24 * squares.sqrt() * 4).all()
