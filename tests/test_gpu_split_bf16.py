"""The split-bf16 transforms where their tiles end, against the FP64 oracle: first-axis bands of one to four blocks of
16, ragged and beyond the split kernels (an axis above 192 runs in FP32), first axes shorter than 64 (the projection
then runs the expansion's kernel), odd and two-tile inner bands, and an inner band above 64 (an axis per kernel); and
a gradient and a Hessian product, which combine and accumulate.  The split keeps 16 bits of an operand (relative error
2^-17 per product, averaged over a contraction); bound 1e-5, as for FP32 trajectories.
"""
import numpy as np
import pytest
import torch

from gpu_common import close, images, oracle_model, velocity
from oracle import spectral as sp
from paper_2006_06823_amd import lddmm_bl as L
from paper_2006_06823_amd import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [((26, 20, 23), (8, 6, 10)), ((70, 18, 34), (18, 8, 12)), ((101, 52, 21), (34, 34, 10)),
                                 ((150, 16, 40), (50, 6, 20)), ((192, 12, 14), (64, 4, 6)), ((200, 20, 18), (40, 8, 6)),
                                 ((40, 18, 200), (12, 6, 66)), ((50, 61), (14, 18))])
def test_transforms(N, K):
    ctx = L.Context(L.Problem(N, K, nt=1, precision=L.BF16_DFT))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=ctx.dtype, device=ctx.device)
    rng = np.random.default_rng(51)
    for nf in (1, 3):
        print(f"N {N} K {K} fields {nf}", flush=True)
        f = rng.standard_normal((nf,) + N).astype(np.float32)
        ref = sp.project(torch.tensor(f, dtype=torch.float64), K)
        got = ctx.project(dev(f if nf > 1 else f[0]), nf)
        assert close(got.reshape(ref.shape), ref, "projection") <= 1e-5
        c = ref.numpy().astype(np.float32)
        grid = sp.include(torch.tensor(c, dtype=torch.float64), N)
        got = ctx.include(dev(c if nf > 1 else c[0]), nf)
        assert close(got.reshape(grid.shape), grid, "inclusion") <= 1e-5


@pytest.mark.parametrize("variant", [L.IMAGE_TRANSPORT, L.DEFORMATION_STATE])
@pytest.mark.parametrize("N,K", [((70, 26, 29), (18, 8, 10)), ((52, 50, 21), (18, 34, 8))])
def test_gradient_and_hessian(N, K, variant):
    I0, I1 = images(N, 52)
    v = velocity(N, K, 2, 53)
    dv = syn.random_bl_coefficients(3, K, 54)
    print(f"N {N} K {K} variant {variant}", flush=True)
    ctx = L.Context(L.Problem(N, K, nt=2, variant=variant, precision=L.BF16_DFT))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device=ctx.device)
    ctx.set_images(dev(I0), dev(I1))
    ctx.state_solve(dev(v))
    g, _ = ctx.adjoint_solve()
    om = oracle_model(variant, N, K, 2, I0, I1)
    om.setup(v)
    om.state()
    om.adjoint()
    assert close(g, om.gradient(), "gradient") <= 1e-5
    assert close(ctx.hess_matvec(dev(dv)), om.hess_matvec(dv), "Hessian product") <= 1e-5
