"""The group search and the column loop of one quantized block against the oracle's exhaustive search,
over the row shapes that steer which candidates are scored: Gaussian and heavy-tailed rows (few
survive the clipping bound), uniform rows (hundreds do: more than the kept batches), one-sided rows,
exact ties, constants, on-grid rows and very small values; groups inside a block, as wide as the
block, streamed past it, of a few columns; every bit width and a grid shorter than the first batch."""
import numpy as np
import pytest

import oracle
from oracle.realq_oracle import QParams, quantize_column

pytestmark = pytest.mark.gpu


def _rows(n, seed):
    r = np.random.default_rng(seed)
    rows = [r.standard_normal(n), r.standard_t(2, n), r.uniform(-1, 1, n), r.uniform(-1, 1, n), r.uniform(0.9, 1, n),
            np.abs(r.standard_normal(n)), -np.abs(r.standard_normal(n)), np.where(r.random(n) < 0.5, -1.0, 1.0),
            np.zeros(n), np.full(n, 0.03125), 2.0 ** -8 * (np.arange(n) % 16 - 5), 1e-30 * r.standard_normal(n),
            np.where(np.arange(n) == n // 2, 100.0, 1e-3 * r.standard_normal(n)), r.laplace(size=n),
            np.repeat(r.standard_normal(-(-n // 2)), 2)[:n], np.round(4 * r.standard_normal(n)) / 8]
    return np.stack(rows).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("bits,group,sym,grid,n", [
    (4, 128, False, 80, 128), (4, 32, False, 80, 128), (4, 1, False, 80, 3), (4, 0, True, 80, 300),
    (4, 0, False, 80, 129), (4, 256, False, 80, 333), (3, 64, False, 100, 192), (2, 128, True, 1, 77),
    (2, 128, False, 80, 65), (4, 128, False, 20, 127),
    # every candidate in one walk: long groups (their last one inside a block), a few columns a group
    (4, 0, False, 80, 700), (3, 0, False, 100, 513), (2, 512, False, 80, 600), (4, 384, False, 20, 900),
    (4, 2, False, 80, 77), (4, 4, False, 100, 66), (3, 1, False, 80, 5)])
def test_search_over_row_shapes(rq, ctx, bits, group, sym, grid, n):
    import torch
    W0 = _rows(n, 31 * bits + n)
    m = W0.shape[0]
    qp = QParams(bits=bits, group=group, sym=sym, grid=grid)
    print(f"[gpu-case] search bits={bits} group={group} sym={sym} grid={grid} n={n}", flush=True)
    gl = group or n
    ng = -(-n // gl)
    W = torch.from_numpy(W0).cuda()
    U = torch.eye(n, device="cuda")  # no compensation: every group is searched on the given values
    codes = torch.empty((m, n), dtype=torch.uint8, device="cuda")
    scales = torch.empty((m, ng), device="cuda")
    zeros = torch.empty((m, ng), dtype=torch.uint8, device="cuda")
    p = rq.qparams(bits=bits, group=group, sym=sym, grid=grid)
    for c0 in range(0, n, 128):
        rq.quantize_block(ctx, W, c0, min(128, n - c0), U, None, p, codes, scales, zeros)
    torch.cuda.synchronize()
    for g in range(ng):
        c = slice(g * gl, min(n, (g + 1) * gl))
        s, z, _ = oracle.realq_oracle.group_search(W0[:, c], qp)[:3]
        s = s.astype(np.float32)
        np.testing.assert_array_equal(zeros[:, g].cpu().numpy(), z)
        np.testing.assert_array_equal(scales[:, g].cpu().numpy(), s)
        q, wh = quantize_column(W0[:, c], s.astype(np.float64)[:, None], z[:, None].astype(np.float64), qp.maxq)
        np.testing.assert_array_equal(codes[:, c].cpu().numpy(), q)
        np.testing.assert_array_equal(W[:, c].cpu().numpy(), wh)
