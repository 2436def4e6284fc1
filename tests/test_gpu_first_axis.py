"""The first-axis kernel and the whole-plane kernels where their tiles end, against the FP64 oracle: first-axis bands in
each of its sizes (up to 16, 32, 48, 64), axes shorter than a chunk, ragged and of several batches of chunks, and odd
inner axes with one and two band tiles.  Tolerances of the other FP32 parity tests: transforms 1e-6, gradients 1e-5.
"""
import numpy as np
import pytest
import torch

from gpu_common import close, images, oracle_model, velocity
from oracle import spectral as sp
from paper_2006_06823_amd import lddmm_bl as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [((3, 21, 23), (2, 8, 10)), ((25, 35, 37), (16, 18, 24)), ((53, 101, 67), (34, 40, 20)),
                                 ((77, 21, 97), (50, 10, 36)), ((201, 19, 99), (64, 12, 64)), ((230, 59, 131), (48, 34, 50))])
def test_transforms(N, K):
    ctx = L.Context(L.Problem(N, K, nt=1, precision=L.FP32))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=ctx.dtype, device=ctx.device)
    rng = np.random.default_rng(61)
    for nf in (1, 3):
        print(f"N {N} K {K} fields {nf}", flush=True)
        f = rng.standard_normal((nf,) + N).astype(np.float32)
        ref = sp.project(torch.tensor(f, dtype=torch.float64), K)
        got = ctx.project(dev(f if nf > 1 else f[0]), nf)
        assert close(got.reshape(ref.shape), ref, "projection") <= 1e-6
        c = ref.numpy().astype(np.float32)
        grid = sp.include(torch.tensor(c, dtype=torch.float64), N)
        got = ctx.include(dev(c if nf > 1 else c[0]), nf)
        assert close(got.reshape(grid.shape), grid, "inclusion") <= 1e-6


@pytest.mark.parametrize("variant", [L.IMAGE_TRANSPORT, L.DEFORMATION_STATE])
@pytest.mark.parametrize("N,K", [((53, 21, 23), (34, 8, 10)), ((27, 31, 35), (18, 10, 24))])
def test_gradient(N, K, variant):
    I0, I1 = images(N, 62)
    v = velocity(N, K, 2, 63)
    print(f"N {N} K {K} variant {variant}", flush=True)
    ctx = L.Context(L.Problem(N, K, nt=2, variant=variant, precision=L.FP32))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=ctx.dtype, device=ctx.device)
    ctx.set_images(dev(I0), dev(I1))
    ctx.state_solve(dev(v))
    g, _ = ctx.adjoint_solve()
    om = oracle_model(variant, N, K, 2, I0, I1)
    om.setup(v)
    om.state()
    om.adjoint()
    assert close(g, om.gradient(), "gradient") <= 1e-5
