"""Nodes displaced by a voxel and more, where the three ways to interpolate them meet, against the FP64 oracle: a few of
them in waves of near ones (1.02 voxels at most), most of them inside their bricks (1.7), and most of them outside,
across the periodic edges (9).  Every tile gives the same bits.  Tolerance: the FP32 trajectory bound of the other
parity tests, 1e-5; a velocity's relative rounding of 3e-7 moves a departure point by 3e-6 of a voxel at most here.
"""
import numpy as np
import pytest
import torch

from gpu_common import close, images, oracle_model, velocity
from paper_2006_06823_amd import lddmm_bl as L
from paper_2006_06823_amd import synthetic as syn

pytestmark = pytest.mark.gpu

NT, K = 2, (4, 6, 4)


@pytest.mark.parametrize("cfl", [1.02, 1.7, 9.0])
@pytest.mark.parametrize("N", [(18, 13, 40), (9, 21, 67)])
def test_far_nodes(N, cfl):
    I0, I1 = images(N, 41)
    v = velocity(N, K, NT, 42, cfl_vox=cfl)
    dv = syn.random_bl_coefficients(3, K, 43)
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")
    for variant in (L.IMAGE_TRANSPORT, L.DEFORMATION_STATE):
        om = oracle_model(variant, N, K, NT, I0, I1)
        om.setup(v)
        om.state()
        om.adjoint()
        ref = [om.Xb, om.Xf, om.m[-1] if variant == 1 else om.m1, om.gradient(), om.hess_matvec(dv)]
        first = None
        try:
            for tile in range(L.tune_candidates("brick")):
                for key in L.brick_tune_keys(N):
                    L.tune_set(key, tile)
                print(f"N {N} cfl {cfl} variant {variant} tile {tile}", flush=True)
                ctx = L.Context(L.Problem(N, K, nt=NT, variant=variant, precision=L.FP32))
                ctx.set_images(dev(I0), dev(I1))
                _, m1 = ctx.state_solve(dev(v), want_m1=True)
                g, _ = ctx.adjoint_solve()
                got = [ctx.get_field(L.FIELD_DEP_BACKWARD), ctx.get_field(L.FIELD_DEP_FORWARD), m1, g,
                       ctx.hess_matvec(dev(dv))]
                torch.cuda.synchronize()
                if first is None:
                    first = got
                    for a, b in zip(got, ref):
                        assert close(a, b) <= 1e-5
                assert all(torch.equal(a, b) for a, b in zip(got, first))
        finally:
            for key in L.brick_tune_keys(N):
                L.tune_set(key, -1)
