"""The grid prefilter at line lengths around its chunk (16 points), its reach (16 points in FP32, 32 in FP64) and
its 16-byte rows, in both precisions, and planes that one workgroup holds, whole or in tiles of 64 columns, or just not.

At a zero velocity a step interpolates at the nodes, where the spline of the prefiltered image is the image: the
final image equals the template.  Tolerance: a pass rounds its output once (unit roundoff u) and has gain at most 3,
so three passes and the 64-tap sum (about 10 u more) stay below 3^3 * 3 u + 10 u, under 100 u.  The adjoint filters
two fields at once, one of them weighted: its gradient against the FP64 oracle, at the bounds of the other parity
tests (1e-5 and 1e-10).
"""
import numpy as np
import pytest
import torch

from gpu_common import close, oracle_model, velocity
from paper_2006_06823_amd import lddmm_bl as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,u,tol", [(L.FP32, 2.0 ** -24, 1e-5), (L.FP64, 2.0 ** -53, 1e-10)])
@pytest.mark.parametrize("N", [(4, 5, 6), (7, 16, 17), (33, 15, 31), (16, 34, 12), (18, 9, 65), (5, 48), (31, 32), (65, 66), (130, 40), (40, 200),
                               (5, 20, 97), (4, 150, 130), (4, 33, 161), (129, 100), (20, 192)])
def test_prefilter_line_lengths(N, precision, u, tol):
    K = (4,) * len(N)
    rng = np.random.default_rng(71)
    I0, I1 = rng.standard_normal(N), rng.standard_normal(N)
    print(f"N {N} precision {precision}", flush=True)
    ctx = L.Context(L.Problem(N, K, nt=1, precision=precision))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=ctx.dtype, device=ctx.device)
    ctx.set_images(dev(I0), dev(I1))
    v = velocity(N, K, 1, 72)
    _, m1 = ctx.state_solve(dev(np.zeros_like(v)), want_m1=True)
    assert close(m1, I0, "node values") <= 100 * u
    ctx.state_solve(dev(v))
    g, _ = ctx.adjoint_solve()
    om = oracle_model(L.IMAGE_TRANSPORT, N, K, 1, I0, I1)
    om.setup(v)
    om.state()
    om.adjoint()
    assert close(g, om.gradient(), "gradient") <= tol
