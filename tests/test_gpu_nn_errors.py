"""A forward pass that runs out of memory leaves no pass to go back through: an error, not a crash, and the network
goes on as before."""
import pytest
import torch

from paper_2006_06823_amd import lddmm_bl as L

pytestmark = pytest.mark.gpu

E_OOM, E_STATE = -2, -5


def test_backward_after_a_forward_without_memory():
    net = L.WarmStartNet(channels=(8, 8), in_size=64, seed=8)
    x = torch.randn(2, 2, 64, 64, 64, device="cuda")
    ref = net.forward(x)
    dout = torch.ones_like(ref)
    B = 1 << 24  # 18 TB of activations
    assert net.lib.lddmm_nn_forward(net.h, x.data_ptr(), B, ref.clone().data_ptr()) == E_OOM
    for b in (2, B):
        assert net.lib.lddmm_nn_backward(net.h, dout.data_ptr(), b) == E_STATE
    assert torch.equal(net.forward(x), ref)
    net.zero_grad()
    net.backward(dout)
    torch.cuda.synchronize()
