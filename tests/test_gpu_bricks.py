"""The interpolation kernels where their window and rows end, against the FP64 oracle.

Rows of every remainder modulo four (the staged and stored quads), grids smaller than a tile, and displacements
of less than a voxel (the window), and of several (the nodes interpolated apart, from the brick and from global
memory).  A node's value depends on neither the tile nor the workgroup that forms it, so the eight tiles agree
bitwise.  Tolerance: the FP32 trajectory bound of the other parity tests, 1e-5.
"""
import numpy as np
import pytest
import torch

from gpu_common import close, images, oracle_model, velocity
from paper_2006_06823_amd import lddmm_bl as L
from paper_2006_06823_amd import synthetic as syn

pytestmark = pytest.mark.gpu

NT = 2


@pytest.mark.parametrize("cfl", [0.8, 3.5])
@pytest.mark.parametrize("N", [(12, 10, 13), (9, 11, 14), (7, 18, 35), (20, 9, 64)])
def test_interpolation_at_row_ends_and_beyond_the_window(N, cfl):
    K = (4, 4, 6)
    I0, I1 = images(N, 31)
    v = velocity(N, K, NT, 32, cfl_vox=cfl)
    dv = syn.random_bl_coefficients(3, K, 33)
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
