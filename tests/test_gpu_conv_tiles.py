"""The convolution kernels at the edges of their tiles, against the FP64 reference network.

Output grids on both sides of the 8, 16 and 32 voxel box widths and not a multiple of any, odd edges (no two
voxels of a row in one load), 1 to 5 tiles of 32 output channels (one to four per workgroup), and input channels
that fill none, one and several groups of 16.  Tolerances: test_gpu_learned's, from the bf16 roundoff of the
operands and the number of contractions a result passes through.
"""
import numpy as np
import pytest
import torch

from oracle import convnet
from test_gpu_learned import _active_biases, _net, _rel, fwd_tol, grad_tol

pytestmark = pytest.mark.gpu

# channels, in_size, batch, out_size
CASES = [((3, 130, 70, 33), 19, 2, 0),   # edges 10, 5, 3, 3
         ((18, 20), 50, 1, 25),          # strides 2, 1 at an odd edge wider than a box
         ((5,), 26, 3, 0),               # one level, stride 1 on two channels
         ((40, 72), 33, 1, 0),           # edges 17, 17
         ((16, 17), 32, 2, 8)]           # strides 2, 2 onto a full small box


@pytest.mark.parametrize("channels,in_size,B,out_size", CASES)
def test_convolutions_at_tile_edges(channels, in_size, B, out_size):
    net = _net(channels, in_size, seed=21, out_size=out_size)
    rng = np.random.default_rng(22)
    x = rng.standard_normal((B, 2, in_size, in_size, in_size)).astype(np.float32)
    params = _active_biases(net.get(0).astype(np.float64), channels, x, in_size, out_size)
    net.set(params.astype(np.float32))
    layers = convnet.make_layers(net.get(0).astype(np.float64), channels, 3, in_size=in_size, out_size=out_size)
    acts = convnet.forward(x, layers)
    xt = torch.from_numpy(x).cuda()
    out = net.forward(xt)
    assert _rel(out.cpu().numpy(), acts[-1]) <= fwd_tol(channels)
    dout = rng.standard_normal(tuple(out.shape)).astype(np.float32)
    net.zero_grad()
    net.backward(torch.from_numpy(dout).cuda())
    g, gref = net.get(1).astype(np.float64), convnet.backward(acts, dout, layers)
    o, cin = 0, 2
    for cout, k3 in [(c, 27) for c in channels] + [(3, 1)]:
        n = cout * cin * k3
        assert _rel(g[o:o + n], gref[o:o + n]) <= grad_tol(channels), ("weights", cout)
        assert _rel(g[o + n:o + n + cout], gref[o + n:o + n + cout]) <= grad_tol(channels), ("bias", cout)
        o += n + cout
        cin = cout
