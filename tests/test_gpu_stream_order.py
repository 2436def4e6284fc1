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


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("N,K", [((24, 20, 28), (8, 6, 10)), ((40, 36), (10, 8))])
def test_products_on_callers_streams(N, K, graphs, monkeypatch):
    """Hessian products enqueued on alternating streams behind their inputs, on more buffer pairs than graphs are
    kept for, and followed at once by calls on the context's stream: all bitwise what a caller who waits gets."""
    if not graphs:
        monkeypatch.setenv("LDDMM_BL_NO_GRAPH", "1")
    ctx = L.Context(L.Problem(N, K, nt=3, precision=L.FP32))
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    I0, I1 = rnd(*N), rnd(*N)
    d = len(N)
    v = ctx.project(0.01 * rnd(d, *N), d)
    dvs = [ctx.project(rnd(d, *N), d) for _ in range(6)]
    ctx.set_images(I0, I1)
    ctx.state_solve(v)
    ref = []
    for x in dvs:
        ref.append(ctx.hess_matvec(x).clone())
        torch.cuda.synchronize()
    E0, _ = ctx.state_solve(v)
    g0, _ = ctx.adjoint_solve()
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), ctx.stream, torch.cuda.Stream()]
    work = torch.randn(2048, 2048, device="cuda")
    torch.cuda.synchronize()
    got = []
    for k in range(18):
        with torch.cuda.stream(streams[k % 4]):
            w = torch.tanh(work @ work)
            x = dvs[k % 6] + 0.0 * w[0, 0]  # written on this stream, behind the product above
            got.append((k % 6, ctx.hess_matvec(x), x))
        if k == 7:
            assert ctx.state_solve(v)[0] == E0
        if k == 11:
            assert torch.equal(ctx.adjoint_solve()[0], g0)
    ctx.close()  # waits for what is still queued
    torch.cuda.synchronize()
    for k, y, x in got:
        assert torch.equal(x, dvs[k]) and torch.equal(y, ref[k]), k
