"""A call reads what the caller's stream has queued, finished or not: inputs written behind a long-running kernel on the
default stream and on another one, and on a stream that is idle."""
import pytest
import torch

from paper_2006_06823_amd import lddmm_bl as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("busy", [True, False])
@pytest.mark.parametrize("other", [True, False])
def test_inputs_queued_on_the_callers_stream(busy, other):
    N, K = (24, 20, 28), (8, 6, 10)
    ctx = L.Context(L.Problem(N, K, nt=1, precision=L.FP32))
    f = torch.randn(N, device="cuda")
    ref = ctx.project(f).clone()
    work = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    s = torch.cuda.Stream() if other else torch.cuda.current_stream()
    for _ in range(5):
        with torch.cuda.stream(s):
            g = torch.zeros(N, device="cuda")
            if busy:
                for _ in range(4):
                    work = torch.tanh(work @ work)
            g.copy_(f)
            assert s.query() is False or not busy
            got = ctx.project(g)
        torch.cuda.synchronize()
        assert torch.equal(got, ref)
