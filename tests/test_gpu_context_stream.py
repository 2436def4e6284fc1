"""Products and the context's stream: a program that has the stream (given, or read from the context) finds products
on it, in order with its own work there; one that has not finds them ordered on the streams it calls from."""
import pytest
import torch

from paper_2006_06823_amd import lddmm_bl as L

pytestmark = pytest.mark.gpu

N, K = (24, 20, 28), (8, 6, 10)


def _solved(n=N, k=K, stream=None):
    ctx = L.Context(L.Problem(n, k, nt=3, precision=L.FP32), stream=stream)
    g = torch.Generator(device="cuda").manual_seed(11)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    d = len(n)
    v = ctx.project(0.01 * rnd(d, *n), d)
    dvs = [ctx.project(rnd(d, *n), d) for _ in range(6)]
    ctx.set_images(rnd(*n), rnd(*n))
    E = ctx.state_solve(v)[0]
    refs = []
    for x in dvs:
        refs.append(ctx.hess_matvec(x))
        torch.cuda.synchronize()
    assert ctx.state_solve(v)[0] == E  # a call that waits: nothing is left on any stream
    return ctx, v, E, dvs, refs


def _busy(s):
    """Some ten milliseconds of work on stream s."""
    with torch.cuda.stream(s):
        w = torch.randn(4096, 4096, device="cuda")
        for _ in range(30):
            w = torch.tanh(w @ w)


@pytest.mark.parametrize("how", ["given", "before", "after", "event"])
def test_stream_covers_a_product(how):
    """The result is there once the context's stream has reached the product, wherever that was called from."""
    ctx, _, _, dvs, refs = _solved(stream=torch.cuda.Stream() if how == "given" else None)
    mine = ctx.stream if how in ("given", "before", "event") else None
    side, third = torch.cuda.Stream(), torch.cuda.Stream()
    out = torch.full_like(refs[0], float("nan"))
    _busy(side)  # warms up
    torch.cuda.synchronize()
    _busy(side)
    with torch.cuda.stream(side):
        ctx.hess_matvec(dvs[0], out)
    mine = mine or ctx.stream
    if how == "event":
        e = torch.cuda.Event()
        e.record(mine)
        third.wait_event(e)
    else:
        mine.synchronize()
    with torch.cuda.stream(third):
        got = out.clone()
    third.synchronize()
    assert torch.equal(got, refs[0])
    torch.cuda.synchronize()


def test_inputs_written_on_the_stream():
    ctx, _, _, dvs, refs = _solved()
    x = torch.zeros_like(dvs[1])
    out = ctx.hess_matvec(x)
    _busy(ctx.stream)  # warms up
    torch.cuda.synchronize()
    _busy(ctx.stream)
    with torch.cuda.stream(ctx.stream):
        x.copy_(dvs[1])
    ctx.hess_matvec(x, out)  # from the default stream, which has nothing queued
    assert torch.equal(out, refs[1])
    torch.cuda.synchronize()


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("n,k", [(N, K), ((40, 36), (10, 8))])
def test_products_of_alternating_streams(n, k, graphs, monkeypatch):
    """No one has the context's stream: products behind their inputs on three streams in turn, on more buffer pairs
    than graphs are kept for, and calls on the context's stream among them."""
    if not graphs:
        monkeypatch.setenv("LDDMM_BL_NO_GRAPH", "1")
    ctx, v, E, dvs, refs = _solved(n, k)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    work = torch.randn(2048, 2048, device="cuda")
    torch.cuda.synchronize()
    got = []
    for i in range(18):
        with torch.cuda.stream(streams[i % 3]):
            w = torch.tanh(work @ work)
            x = dvs[i % 6] + 0.0 * w[0, 0]  # written on this stream, behind the product above
            got.append((i % 6, ctx.hess_matvec(x), x))
        if i % 7 == 4:
            assert ctx.state_solve(v)[0] == E
    ctx.close()  # waits for what is still queued
    torch.cuda.synchronize()
    for i, y, x in got:
        assert torch.equal(x, dvs[i]) and torch.equal(y, refs[i]), i
