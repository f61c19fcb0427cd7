"""The token contractions accumulated in float64 (Hessian, Fisher) at the edges of their tiles and token
splits, onto a nonzero accumulator, against float64: one 256-wide tile and less, ragged last tiles,
tokens below a split, ragged in the 32-token slices, unaligned rows (odd n), many splits, few enough
tokens to go straight into the matrix (unweighted, one tile row or eight and more).  Products
of bf16 values are exact and at most L of them are summed in float32 (1024 in a slice of the two high
terms of a weighted product, a staged chunk in the allocation-free call, else at most all T), so an
entry is off by at most (L + 2) 2^-24 of its sum of absolute values (the 2 covers the weighted
operand's rounding; the third term, 2^-17 of the product, is summed over at most T tokens).  Norm-wise
each matrix instruction's 16 products round once, by 2^-24 / sqrt(3) rms of a partial sum that is no
larger than the whole: (sqrt(2 L / 16) + 2) 2^-24 / sqrt(3) with two passes over the terms."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n,T", [(1, 1), (5, 33), (64, 700), (255, 4000), (256, 300), (257, 1031), (520, 20000),
                                 (1030, 2056), (2100, 300)])
def test_accumulated_products_at_tile_edges(rq, ctx, n, T, weighted):
    import torch
    print(f"[gpu-case] accumulated products n={n} T={T} weighted={weighted}", flush=True)
    g = torch.Generator().manual_seed(7 * n + T)
    X = (torch.randn((T, n), generator=g) * 2).to(torch.bfloat16)
    s = torch.exp(2 * torch.randn(T, generator=g)) if weighted else None
    X64 = X.double()
    sx = X64 if s is None else X64 * s.double()[:, None]
    H0 = torch.randn((n, n), generator=g, dtype=torch.float64)
    H0 = H0 + H0.T
    ref, bound = H0 + sx.T @ X64, sx.abs().T @ X64.abs()
    outs = []
    for fn in (rq.hessian_accum, rq.hessian_accum_noalloc):
        H = H0.cuda()
        fn(ctx, X.cuda(), None if s is None else s.cuda(), H)
        torch.cuda.synchronize()
        outs.append(H.cpu())
    staged = (16 << 20) // (2 * n) // 256 * 256  # tokens per chunk of the allocation-free call
    for H, most in zip(outs, (1024 if weighted else T, staged)):
        L = min(T, most)
        assert bool(((H - ref).abs() <= (L + 2 + T * 2.0 ** -16) * 2.0 ** -24 * bound + 1e-12).all())
        rel = float((H - ref).norm() / (ref - H0).norm())
        print("norm-wise", rel, "of", (np.sqrt(L / 8) + 2) * 2.0 ** -24 / np.sqrt(3), flush=True)
        assert rel <= (np.sqrt(L / 8) + 2) * 2.0 ** -24 / np.sqrt(3)
    assert torch.equal(outs[0], outs[0].T)  # one triangle is formed
    if not weighted:
        F = H0.cuda()
        rq.fisher_accum(ctx, X.cuda(), F)
        assert torch.equal(F.cpu(), outs[0])


@pytest.mark.parametrize("n,T,dominant", [(520, 20000, False), (520, 20000, True), (1030, 6500, True),
                                          (7001, 18501, False)])
def test_weighted_sums_over_many_slices(rq, ctx, n, T, dominant):
    """Weighted sums over many slices of at most 1024 tokens and (7001 columns) over two panels of rows,
    norm-wise against float64, also where three tokens carry the sums.  A slice adds 1024 / 16 matrix
    instructions' products for each of the two high terms, each rounding by 2^-24 / sqrt(3) rms at most:
    sqrt(128) 2^-24 / sqrt(3) = 3.9e-7 (measured 6e-8 to 2.1e-7).  Without the third bf16 term of s x the
    error is 6.4e-7 to 2.5e-6, which the reference shows on its own sums."""
    import torch
    print(f"[gpu-case] weighted sums n={n} T={T} dominant={dominant}", flush=True)
    g = torch.Generator().manual_seed(n + T)
    X = (torch.randn((T, n), generator=g) * 2).to(torch.bfloat16).cuda()
    s = torch.exp(torch.randn(T, generator=g))
    if dominant:
        s[torch.randperm(T, generator=g)[:3]] *= 1e5
    s = s.cuda()
    H = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    rq.hessian_accum(ctx, X, s, H)
    ref, two = torch.zeros_like(H), torch.zeros_like(H)
    for t in range(0, T, 4096):
        x, w = X[t:t + 4096], s[t:t + 4096, None]
        sx = x.float() * w
        hi = sx.bfloat16().float()
        lo = (sx - hi).bfloat16()
        ref += (x.double() * w.double()).T.contiguous() @ x.double()
        two += (hi.double() + lo.double()).T.contiguous() @ x.double()
    assert torch.equal(H, H.T)
    assert float((H - ref).norm()) <= 4e-7 * float(ref.norm()) < float((two - ref).norm())
