"""The transforms' half-plane kernels (a band above 32 on an even inner axis) where their tiles and pairs end, against
the FP64 oracle: bands that are no multiple of 4 or above 48, one axis above 32 and the other not, half axes that
are odd, shorter than a tile or just beyond one; and through gradient and Hessian product, whose reductions form
products of several fields.  Tolerances of the other FP32 parity tests: transforms 1e-6, gradients and products 1e-5.
"""
import numpy as np
import pytest
import torch

from gpu_common import close, images, oracle_model, velocity
from oracle import spectral as sp
from paper_2006_06823_amd import lddmm_bl as L
from paper_2006_06823_amd import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [((6, 50, 20), (4, 34, 6)), ((5, 20, 54), (4, 8, 36)), ((4, 98, 100), (2, 64, 62)),
                                 ((3, 130, 66), (2, 50, 42)), ((7, 62, 128), (4, 40, 48)), ((2, 194, 258), (2, 64, 34))])
def test_transforms(N, K):
    ctx = L.Context(L.Problem(N, K, nt=1, precision=L.FP32))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=ctx.dtype, device=ctx.device)
    rng = np.random.default_rng(91)
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
@pytest.mark.parametrize("N,K", [((12, 52, 58), (4, 34, 36)), ((10, 66, 32), (4, 42, 10))])
def test_gradient_and_hessian(N, K, variant):
    I0, I1 = images(N, 92)
    v = velocity(N, K, 2, 93)
    dv = syn.random_bl_coefficients(3, K, 94)
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
    assert close(ctx.hess_matvec(dev(dv)), om.hess_matvec(dv), "Hessian product") <= 1e-5
