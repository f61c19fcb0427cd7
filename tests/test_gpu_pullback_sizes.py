"""The pulled-back metric P = W^T M W at tile edges and odd sizes, in float64 where it is small (up to
512 rows, or 1024 with a dense M) and in bf16 terms above, for bf16-exact and full float32
weights (the lower terms of an exact weight are skipped), with and without a (non-symmetric) M,
stored and accumulated, against float64.  Three bf16 terms carry all 24 bits and the dropped term
pairs are below 2^-25 of the product; sums of K float32 products round by at most K 2^-24 of the sum
of absolute values (twice, with M, whose inner product is rounded to float32 once more).  That
bounds every entry at any size; what a lost term leaves is checked norm-wise below."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("m_next,m,dense", [(1, 1, False), (37, 65, False), (300, 257, False), (1023, 520, False),
                                            (513, 65, False), (700, 257, False), (256, 2049, False),
                                            (65, 37, True), (264, 300, True), (1030, 37, True), (1025, 257, True)])
def test_pullback_at_tile_edges(rq, ctx, m_next, m, dense, exact, accumulate):
    import torch
    print(f"[gpu-case] pullback {m_next}x{m} dense={dense} exact={exact} accumulate={accumulate}", flush=True)
    g = torch.Generator().manual_seed(m_next + 3 * m)
    W = torch.randn((m_next, m), generator=g)
    if exact:
        W = W.to(torch.bfloat16).float()
    M = torch.randn((m_next, m_next), generator=g) if dense else None
    P0 = torch.randn((m, m), generator=g)
    P = P0.cuda()
    rq.pullback_metric(ctx, W.cuda(), P, None if M is None else M.cuda(), accumulate=accumulate)
    torch.cuda.synchronize()
    W64 = W.double()
    R = W64 if M is None else M.double() @ W64
    Ra = W64.abs() if M is None else M.double().abs() @ W64.abs()
    ref = W64.T @ R + (P0.double() if accumulate else 0.0)
    bound = (2 * m_next + 6) * 2.0 ** -24 * (W64.abs().T @ Ra) + 2.0 ** -23 * (ref.abs() + P0.double().abs())
    assert bool(((P.cpu().double() - ref).abs() <= bound).all())
    if not dense and not accumulate:
        assert torch.equal(P, P.T)


@pytest.mark.parametrize("m_next,m,dense,accumulate", [(1023, 520, False, False), (1100, 520, True, True),
                                                       (4000, 300, False, True), (515, 14500, False, True),
                                                       (300, 14500, True, False)])
def test_pullback_of_full_float32_weights(rq, ctx, m_next, m, dense, accumulate):
    """Norm-wise, where a lost term shows, and over several panels of rows (14500 columns): sums of at
    most 1024 products in 64 matrix instructions a pass round by sqrt(128) 2^-24 / sqrt(3) = 3.9e-7 rms at
    most (measured 4e-8 to 1.5e-7); two bf16 terms instead of three leave 9e-7 to 3.5e-6."""
    import torch
    print(f"[gpu-case] pullback, three terms {m_next}x{m} dense={dense}", flush=True)
    g = torch.Generator().manual_seed(m_next + 3 * m)
    W = torch.randn((m_next, m), generator=g).cuda()
    M = torch.randn((m_next, m_next), generator=g).cuda() if dense else None
    P0 = torch.randn((m, m), generator=g).cuda()
    P = P0.clone()
    rq.pullback_metric(ctx, W, P, M, accumulate=accumulate)
    hi = W.bfloat16().float()

    def product(w):
        r = w if M is None else M.double() @ w
        return w.T.contiguous() @ r + (P0.double() if accumulate else 0.0)

    ref, two = product(W.double()), product(hi.double() + (W - hi).bfloat16().double())
    assert float((P.double() - ref).norm()) <= 4e-7 * float(ref.norm()) < float((two - ref).norm())
    if not dense and not accumulate:
        assert torch.equal(P, P.T)
