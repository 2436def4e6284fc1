"""Calls that only enqueue and a caller's stream captures: beside one, and within one after products on other streams.
Replays follow the context's own eager calls and are compared with them bit by bit."""
import threading

import pytest
import torch

from paper_2006_06823_amd import lddmm_bl as L

pytestmark = pytest.mark.gpu


def _solved(N, K):
    """A context at a solved state, its inputs, and a product behind it on a stream of its own (the usual warm-up)."""
    ctx = L.Context(L.Problem(N, K, nt=3, precision=L.FP32))
    g = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    d = len(N)
    v = ctx.project(0.01 * rnd(d, *N), d)
    dv = ctx.project(rnd(d, *N), d)
    ctx.set_images(rnd(*N), rnd(*N))
    ctx.state_solve(v)
    out = torch.empty_like(dv)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ctx.hess_matvec(dv, out)
    torch.cuda.synchronize()
    return ctx, rnd, dv, out, side


@pytest.mark.parametrize("thread", [False, True])
def test_calls_beside_a_capture(thread):
    """A capture of other work runs on this thread, and the calls come from a stream that it does not capture."""
    N, K = (24, 20, 28), (8, 6, 10)
    ctx, rnd, dv, out, side = _solved(N, K)
    ref = out.clone()
    f, bl = rnd(N[0], N[1], N[2]), torch.zeros(K, device="cuda")
    ctx.project_noalloc(f, bl)  # the first call looks the library's workspace up
    bl_ref = bl.clone()
    x = torch.ones(8, device="cuda")
    torch.cuda.synchronize()
    failed = []

    def calls():
        try:
            with torch.cuda.stream(side):
                for t in (bl, out):
                    t.fill_(float("nan"))
                ctx.project_noalloc(f, bl)
                ctx.hess_matvec(dv, out)
        except Exception as e:
            failed.append(e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y = x * 2
        if thread:
            t = threading.Thread(target=calls)
            t.start()
            t.join()
        else:
            calls()
    assert not failed
    torch.cuda.synchronize()
    assert torch.equal(bl, bl_ref) and torch.equal(out, ref)
    for i in range(3):
        x.fill_(float(i))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, x * 2)
