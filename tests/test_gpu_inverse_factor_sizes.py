"""The inverse factor at the edges of its panels and tiles (64-wide panels, outer panels of 256, 128-wide
trailing and doubling tiles once they fill the chip, padded last panels and cut-off last pairs), each
size twice on one context with different Hessians: the work arrays of a call hold the previous call's
values.  Float64 throughout, so U may differ from the oracle's by its float32 rounding (2^-24 relative)
plus the factorisation's own rounding, about n 2^-53 cond(H_d) <= 4100 * 1.1e-16 * 1e4 = 4.5e-9."""
import numpy as np
import pytest

import oracle
from oracle.realq_oracle import damp_hessian, inverse_factor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129, 256, 257, 320, 1000, 4100])
def test_inverse_factor_at_tile_edges(rq, ctx, n):
    import torch
    print(f"[gpu-case] inverse factor n={n}", flush=True)
    r = np.random.default_rng(n)
    T = 2 * n + 3
    for _ in range(2):
        X = torch.from_numpy(r.standard_normal((T, n)) * (1 + 3 * (r.random(n) < 0.05)))
        H = (X.T @ X).numpy()
        U = torch.empty((n, n), device="cuda")
        Hout = torch.empty((n, n), device="cuda")
        rq.chol_inverse(ctx, torch.from_numpy(H).cuda(), T, 0.01, U, Hout)
        torch.cuda.synchronize()
        Hs = H * (2.0 / T)
        np.testing.assert_array_equal(Hout.cpu().numpy(), Hs.astype(np.float32))
        ref = inverse_factor(damp_hessian(Hs, float(np.float32(0.01)))[0])
        got = U.cpu().numpy().astype(np.float64)
        assert np.array_equal(got, np.triu(got))
        assert np.abs(got - ref).max() <= (2.0 ** -24 + 1e-8) * np.abs(ref).max()
