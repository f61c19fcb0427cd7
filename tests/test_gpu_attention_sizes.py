"""The attention forward at its edges: one, three and five key tiles (a block takes four query
tiles), head widths with their own kernels (64, 128) and without (96), scores from nearly uniform to
so wide that the running maximum keeps moving and most probabilities vanish."""
import numpy as np
import pytest

import synth
from oracle import block_oracle as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spread", [0.05, 30.0])
@pytest.mark.parametrize("hd,L", [(128, 32), (128, 160), (64, 96), (96, 160)])
def test_attention_forward(rq, ctx, hd, L, spread):
    import torch
    H, Hkv, T, d = 4, 2, 3 * L, 64
    inp = synth.make_decoder_block(T, d, 64, H, Hkv, hd, L, seed=hd + L, dense_F=False)
    w = {k: None if v is None else torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).cuda()
         for k, v in inp.w.items()}
    gen = np.random.default_rng(3)
    for k, n in (("Wq", H), ("Wk", Hkv)):  # q . k / sqrt(hd) of about this spread
        w[k] = torch.from_numpy((gen.standard_normal((n * hd, d)) * np.sqrt(spread / d)).astype(np.float32)).cuda()
    print(f"[gpu-case] attention forward hd={hd} L={L} spread={spread}", flush=True)
    r = rq.decoder_forward(ctx, torch.from_numpy(inp.X.astype(np.float32)).cuda().bfloat16(), w, n_heads=H, n_kv=Hkv,
                           head_dim=hd, seq_len=L, intermediates=True)
    torch.cuda.synchronize()
    q, k, v, O = (r[x].float().cpu().numpy().astype(np.float64) for x in ("q", "k", "v", "O"))
    ref, P = B.attention_forward(B.bf16(B.rope(q, H, hd, L)), B.bf16(B.rope(k, Hkv, hd, L)), v, H, Hkv, hd, L)
    # bf16 rounds each entry of O by at most 2^-9 of it; as much again for a rotated q or k whose
    # rounding falls the other way
    assert np.isfinite(O).all()
    assert np.linalg.norm(O - ref) <= 2.0 ** -8 * np.linalg.norm(ref)
    assert float((O != B.bf16(ref)).mean()) <= 3e-3
