"""Padded operand layouts of the Block-GD state: odd columns (rows padded to 16 bytes), odd token
counts, and token chunks or mini-batches that do not start on multiples of 8 tokens (each chunk then
has its own padded place, or, where chunks are short, the tokens keep their order), with weights, the
clip, increments, a metric, a window partner and row groups, against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,T,batch,chunk,clip", [
    (37, 133, 1003, 0, 0, 0.0), (37, 133, 1003, 0, 101, 0.0), (37, 136, 1003, 333, 0, 0.0),
    (37, 133, 1003, 335, 97, 0.0), (40, 133, 1003, 336, 96, 0.0), (37, 133, 1003, 335, 97, 0.95),
    (37, 133, 1003, 0, 13, 0.0), (37, 136, 1003, 9, 0, 0.0), (37, 133, 1003, 100, 33, 0.95),
    (300, 260, 517, 0, 0, 0.95)])
def test_ragged_layouts(rq, ctx, m, n, T, batch, chunk, clip):
    import torch
    print(f"[gpu-case] ragged layout m={m} n={n} T={T} batch={batch} chunk={chunk} clip={clip}", flush=True)
    L = synth.make_module("qwen3_0.6b_mlp", m=m, n=n, T=T)
    W0, X, Xh, s, _ = P.to_device(L, torch)
    lr, steps = 1e-5, 3
    g = rq.quantize_layer(ctx, W0, X, Xh, s, qp=rq.qparams(),
                          bgd=rq.bgd_params(steps=steps, lr=lr, batch=batch, tok_chunk=chunk, loss_clip=clip))
    o = oracle.quantize_layer(L.W0, L.X, L.Xhat, L.s, steps=steps, lr=lr, batch=batch or None,
                              loss_clip=clip or None)
    met = P.compare(g, o)
    assert met["code_identity"] >= P.CODE_IDENTITY, met
    assert abs(g.loss_final - o.loss_final) <= P.LOSS_RTOL * abs(o.loss_final)
    tr = g.loss_trace.cpu().numpy()[:steps]
    np.testing.assert_allclose(tr, [v for (_, _, v) in o.loss_trace][:steps], rtol=1e-4)


@pytest.mark.parametrize("option", ["increments", "metric", "window", "row_groups"])
@pytest.mark.parametrize("batch,chunk", [(0, 101), (0, 13), (1103, 0)])
def test_token_places_with(rq, ctx, option, batch, chunk):
    """Chunks and batches off the multiples of 8 (13-token chunks keep the tokens' order) together
    with what else a step can hold; 16 tokens per column and the workload's lr, so the full-batch
    cases take increments."""
    import torch
    print(f"[gpu-case] token places with {option} batch={batch} chunk={chunk}", flush=True)
    L = synth.make_module("llama3.1_8b_layer", "q", m=72, n=133, T=2203, seed=21)
    r = np.random.default_rng(22)
    M = Pm = S = window = None
    if option == "metric":
        A = r.standard_normal((72, 144))
        M = (A @ A.T / 144).astype(np.float32)
    elif option == "window":
        Pm = oracle.pullback_metric((r.standard_normal((50, 72)) * 0.05).astype(np.float32)).astype(np.float32)
        window = (1, 3)
    elif option == "row_groups":
        S = synth.make_group_weights(3, 2203, seed=23)
    W0, X, Xh, s, _ = P.to_device(L, torch)
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()  # noqa: E731
    res = {}
    for inc in (1, 0):
        res[inc] = rq.quantize_layer(ctx, W0, X, Xh, s, dev(M), dev(Pm), qp=rq.qparams(), window=window, s_groups=dev(S),
                                     bgd=rq.bgd_params(steps=4, lr=L.lr, batch=batch, tok_chunk=chunk,
                                                       resid_increment=inc))
    torch.cuda.synchronize()
    o = oracle.quantize_layer(L.W0, L.X, L.Xhat, L.s, M=M, P=Pm, steps=4, lr=L.lr, window=window, batch=batch or None,
                              s_groups=S)
    for g in res.values():
        met = P.compare(g, o)
        assert met["code_identity"] >= P.CODE_IDENTITY, met
        assert abs(g.loss_final - o.loss_final) <= P.LOSS_RTOL * abs(o.loss_final)
    same = res[1].loss_final == res[0].loss_final and bool((res[1].W_hat == res[0].W_hat).all())
    assert same == bool(batch)  # increments are taken with the full batch only
