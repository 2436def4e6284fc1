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


@pytest.mark.parametrize("N,K", [((24, 20, 28), (8, 6, 10)), ((64, 48, 40), (16, 12, 16))])
def test_projection_captured_after_a_product(N, K):
    ctx, rnd, dv, out, side = _solved(N, K)
    ref = out.clone()
    f, bl = torch.zeros(N, device="cuda"), torch.zeros(K, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.project_noalloc(f, bl)
    for _ in range(4):
        f.copy_(rnd(*N))
        bl.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(bl, ctx.project(f))
        assert torch.equal(ctx.hess_matvec(dv), ref)  # and the products after it are as before
        torch.cuda.synchronize()


@pytest.mark.parametrize("N,K", [((24, 20, 28), (8, 6, 10)), ((40, 36), (10, 8))])
def test_product_captured_after_a_product(N, K, monkeypatch):
    monkeypatch.setenv("LDDMM_BL_NO_GRAPH", "1")  # the launches themselves are captured
    ctx, rnd, dv, out, side = _solved(N, K)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.hess_matvec(dv, out)
    for _ in range(4):
        dv.copy_(ctx.project(rnd(len(N), *N), len(N)))
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        with torch.cuda.stream(side):
            side.wait_stream(torch.cuda.default_stream())
            eager = ctx.hess_matvec(dv)
        torch.cuda.synchronize()
        assert torch.equal(got, eager)


def test_capture_does_not_take_the_wait_of_later_calls():
    """A capture begun while a product still runs: the call after it on the context's stream waits for the product."""
    ctx, rnd, dv, out, side = _solved((24, 20, 28), (8, 6, 10))
    ref = out.clone()
    v2 = ctx.project(0.01 * rnd(3, 24, 20, 28), 3)
    f, bl = rnd(24, 20, 28), torch.zeros(8, 6, 10, device="cuda")
    work = torch.randn(4096, 4096, device="cuda")
    ctx.project_noalloc(f, bl)
    torch.cuda.synchronize()
    out.fill_(float("nan"))
    torch.cuda.synchronize()
    capture = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        for _ in range(30):
            work = torch.tanh(work @ work)
        ctx.hess_matvec(dv, out)
    with torch.cuda.stream(capture):
        graph.capture_begin()
        ctx.project_noalloc(f, bl)
        graph.capture_end()
    assert not side.query()
    ctx.state_solve(v2)  # overwrites the state that the product reads
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


def test_product_on_a_captured_stream_is_refused():
    """The C call, which the binding keeps from streams under capture; the capture goes on."""
    N, K = (24, 20, 28), (8, 6, 10)
    ctx, rnd, dv, out, side = _solved(N, K)
    ref = out.clone()
    f, bl = rnd(*N), torch.zeros(K, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cur = torch.cuda.current_stream()
        st = ctx.lib.lddmm_bl_hess_matvec_on(ctx.h, dv.data_ptr(), out.data_ptr(), cur.cuda_stream)
        ctx.project_noalloc(f, bl)  # from here the context's stream is under capture as well
        st2 = ctx.lib.lddmm_bl_hess_matvec_on(ctx.h, dv.data_ptr(), out.data_ptr(), side.cuda_stream)
    assert st == st2 == -5  # E_STATE
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(bl, ctx.project(f))
    assert torch.equal(ctx.hess_matvec(dv), ref)
