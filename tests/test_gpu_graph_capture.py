"""Calls recorded into a graph after a larger call on the same context (nothing may be allocated then),
replayed with eager work and synchronizations in between, bitwise as the eager call."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["hessian", "hessian_weighted", "pullback", "pullback_dense", "handoff_odd"])
def test_replays_match_the_eager_call(rq, call):
    import torch
    print(f"[gpu-case] graph capture of {call}", flush=True)
    g = torch.Generator().manual_seed(11)
    stream = torch.cuda.Stream()

    def inputs(T, n, m):
        r = lambda *s: torch.randn(s, generator=g).cuda()  # noqa: E731
        return dict(X=r(T, n).bfloat16(), s=torch.exp(r(T)), H=torch.zeros((n, n), dtype=torch.float64, device="cuda"),
                    W=r(m, n), M=r(m, m), P=torch.zeros((n, n), device="cuda"),
                    Y=torch.zeros((T, m), dtype=torch.bfloat16, device="cuda"))

    def run(ctx, a):
        if call.startswith("hessian"):
            a["H"].zero_()
            rq.hessian_accum(ctx, a["X"], a["s"] if call.endswith("weighted") else None, a["H"])
            return a["H"]
        if call.startswith("pullback"):
            rq.pullback_metric(ctx, a["W"], a["P"], a["M"] if call.endswith("dense") else None)
            return a["P"]
        rq.handoff(ctx, a["W"], a["X"], a["Y"])
        return a["Y"]

    big, small = inputs(5000, 1544, 1100), inputs(3001, 517, 300)
    with torch.cuda.stream(stream):
        ctx = rq.Context(stream)
        run(ctx, big)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            out = run(ctx, small)
        for i in range(4):
            out.fill_(float(i))
            graph.replay()
            stream.synchronize()
            got = out.clone()
            torch.randn(1 << 16, device="cuda").sum().item()
            assert torch.equal(got, run(ctx, small)), i
        stream.synchronize()
        ctx.close()
