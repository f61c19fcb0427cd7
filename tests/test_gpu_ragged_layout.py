"""Padded operand layouts of the Block-GD state: odd columns (rows padded to 16 bytes), odd token
counts, and token chunks or mini-batches that do not start on multiples of 8 tokens (each chunk then
has its own padded place), with weights and with the clip, against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,T,batch,chunk,clip", [
    (37, 133, 1003, 0, 0, 0.0), (37, 133, 1003, 0, 101, 0.0), (37, 136, 1003, 333, 0, 0.0),
    (37, 133, 1003, 335, 97, 0.0), (40, 133, 1003, 336, 96, 0.0), (37, 133, 1003, 335, 97, 0.95),
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
