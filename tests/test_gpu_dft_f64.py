"""The FP64 transforms where their tiles end, against the oracle: bands and axes that are no multiple of 4 or 16, of
one, two, three and four 16-row tiles, beyond the fused kernels (a band above 64, a plane above 256 x 256), in two
and three dimensions, for several fields; and a gradient and a Hessian product, which combine, scale and accumulate.
Tolerance 1e-10, that of the other FP64 parity tests.
"""
import numpy as np
import pytest
import torch

from gpu_common import close, images, oracle_model, velocity
from oracle import spectral as sp
from paper_2006_06823_amd import lddmm_bl as L
from paper_2006_06823_amd import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [((5, 6), (2, 4)), ((37, 50), (14, 18)), ((64, 61), (16, 20)), ((130, 97), (40, 34)),
                                 ((67, 140), (22, 64)), ((150, 40), (66, 12)), ((48, 230), (10, 70)),
                                 ((300, 260), (20, 12)), ((9, 20, 33), (4, 6, 18)), ((20, 12, 150), (6, 4, 66))])
def test_transforms(N, K):
    ctx = L.Context(L.Problem(N, K, nt=1, precision=L.FP64))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=ctx.dtype, device=ctx.device)
    rng = np.random.default_rng(81)
    for nf in (1, 3):
        print(f"N {N} K {K} fields {nf}", flush=True)
        f = rng.standard_normal((nf,) + N)
        ref = sp.project(torch.tensor(f), K)
        got = ctx.project(dev(f if nf > 1 else f[0]), nf)
        assert close(got.reshape(ref.shape), ref, "projection") <= 1e-10
        grid = sp.include(ref, N)
        got = ctx.include(dev(ref.numpy() if nf > 1 else ref.numpy()[0]), nf)
        assert close(got.reshape(grid.shape), grid, "inclusion") <= 1e-10


@pytest.mark.parametrize("variant", [L.IMAGE_TRANSPORT, L.DEFORMATION_STATE])
@pytest.mark.parametrize("N,K", [((37, 50), (14, 18)), ((40, 33), (6, 16)), ((12, 18, 21), (4, 6, 8))])
def test_gradient_and_hessian(N, K, variant):
    I0, I1 = images(N, 82)
    v = velocity(N, K, 3, 83)
    dv = syn.random_bl_coefficients(len(N), K, 84)
    print(f"N {N} K {K} variant {variant}", flush=True)
    ctx = L.Context(L.Problem(N, K, nt=3, variant=variant, precision=L.FP64))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=ctx.dtype, device=ctx.device)
    ctx.set_images(dev(I0), dev(I1))
    ctx.state_solve(dev(v))
    g, _ = ctx.adjoint_solve()
    om = oracle_model(variant, N, K, 3, I0, I1)
    om.setup(v)
    om.state()
    om.adjoint()
    assert close(g, om.gradient(), "gradient") <= 1e-10
    assert close(ctx.hess_matvec(dev(dv)), om.hess_matvec(dv), "Hessian product") <= 1e-10
