// Host-side launch planning of the layer sweep (see plan.h).
#include "plan.h"

#include <algorithm>

namespace realq {
namespace plan {

int64_t tiles(int64_t M, int64_t N, bool large) {
    const int64_t bm = large ? kLargeBM : kSmallBM, bn = large ? kLargeBN : kSmallBN;
    return ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
}

bool pick_large(int64_t M, int64_t N, int tile) {
    return tile == 1 || (tile == 0 && tiles(M, N, true) >= kLargeMinTiles);
}

int64_t num_blocks(int64_t M, int64_t N, int tile) { return tiles(M, N, pick_large(M, N, tile)); }

int64_t k_per_split(int64_t K, int64_t splits) {
    if (splits < 1) splits = 1;
    int64_t kps = (K + splits - 1) / splits;
    kps = ((kps + kBK - 1) / kBK) * kBK;
    return kps <= 0 ? kBK : kps;
}

int64_t effective_splits(int64_t K, int64_t splits) {
    const int64_t kps = k_per_split(K, splits);
    const int64_t s = (K + kps - 1) / kps;
    return s < 1 ? 1 : s;
}

int64_t choose_splits(int64_t M, int64_t N, int64_t K, int cus) {
    if (cus < 1) cus = 1;
    const int64_t blocks = tiles(M, N, true);
    int64_t smax = std::min<int64_t>(16, K / 256);
    if (smax < 1) smax = 1;
    int64_t best = 1;
    double best_fill = -1.0;
    for (int64_t q = 1; q <= smax; ++q) {
        const int64_t bq = blocks * q;
        const int64_t rounds = (bq + cus - 1) / cus;
        const double fill = (double)bq / (double)(rounds * cus);
        if (fill >= 0.97) return q;
        if (fill > best_fill + 1e-9) {
            best_fill = fill;
            best = q;
        }
    }
    return best;
}

int64_t row_stride(int64_t n) { return (n + 63) / 64 * 64; }

int64_t operand_stride(int64_t n) {
    const int64_t lines = (n + 63) / 64;
    return 64 * (lines | 1);
}

bool pullback_small(int64_t m_next, int64_t m, bool dense) {
    const double mm = (double)m * (double)m;
    if (!dense) return m_next <= 512 && mm * (double)m_next <= 0x1p30;
    // 35 ns per 10^6 products in float64, 12 in six bf16 passes; what the launches and slices cost there
    return m_next <= 1024 && 2.3e-8 * (double)m * (double)m_next * (double)(m_next + m) <= 130.0 + 8e-6 * mm;
}

bool straight_acc(int64_t M, int64_t K, int cus) {
    if (cus < 1) cus = 1;
    const int64_t nt = (M + kLargeBM - 1) / kLargeBM, half = nt * (nt + 1) / 2;
    if (nt > 1 && nt < 8) return false;
    const int64_t extra = (nt * nt + cus - 1) / cus - (half + cus - 1) / cus;
    return (double)extra * (double)K * 0.030 <= 0.21 * (double)half;
}

int64_t panel_rows(int64_t M, int64_t N, bool symmetric, int64_t slices, int64_t r0, int64_t budget) {
    int64_t lo = 1, hi = (M - r0 + kLargeBM - 1) / kLargeBM;  // tiles
    if (panel_bytes(N, symmetric, slices, r0, M - r0) <= budget) return M - r0;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (panel_bytes(N, symmetric, slices, r0, std::min(mid * kLargeBM, M - r0)) <= budget) lo = mid;
        else hi = mid - 1;
    }
    return std::min(lo * kLargeBM, M - r0);
}

int64_t even_budget(int64_t M, int64_t N, bool symmetric, int64_t slices, int64_t budget) {
    auto panels = [&](int64_t b) {
        int64_t k = 0;
        for (int64_t r0 = 0; r0 < M; ++k) r0 += panel_rows(M, N, symmetric, slices, r0, b);
        return k;
    };
    const int64_t k = panels(budget);
    if (k == 1) return budget;
    int64_t lo = 0, hi = budget;
    while (hi - lo > budget / 100) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (panels(mid) <= k) hi = mid;
        else lo = mid;
    }
    return hi;
}

Places place_tokens(int64_t T, int64_t Tb, int64_t Tc, bool may_part) {
    Places L;
    L.T = T;
    L.Tb = L.batch = Tb;
    L.Tc = L.chunk = Tc;
    L.count = T;
    if (!may_part || ((Tc >= T || Tc % 8 == 0) && (Tb >= T || Tb % 8 == 0))) return L;
    auto round8 = [](int64_t v) { return (v + 7) / 8 * 8; };
    Places P = L;
    P.apart = true;
    P.chunk = round8(Tc);
    P.batch = Tb / Tc * P.chunk + round8(Tb % Tc);
    P.count = place_of(P, T - 1) + 1;
    return P.count <= T + T / 16 ? P : L;
}

int64_t choose_acc_splits(int64_t tiles, int64_t K, int passes, int cus, int64_t max_k) {
    if (cus < 1) cus = 1;
    const int64_t smin = max_k > 0 ? (K + max_k - 1) / max_k : 1;
    const int64_t smax = std::max<int64_t>(smin, std::min<int64_t>(256, K / 256));
    int64_t best = smin;
    double best_cost = 0.0;
    for (int64_t q = smin; q <= smax; ++q) {
        const int64_t rounds = (tiles * q + cus - 1) / cus;
        const double cost = (double)rounds * (double)K / (double)q * 0.030 * passes + 0.11 * (double)(tiles * q);
        if (q == smin || cost < best_cost) {
            best = q;
            best_cost = cost;
        }
    }
    return effective_splits(K, best);
}

StepPlan plan_step(int64_t m, int64_t nJ, int64_t T, int64_t Tb, int64_t Tc, int64_t t, int cus,
                   int64_t clip_parts) {
    StepPlan p;
    if (Tb < 1 || Tb > T) Tb = T;
    if (Tc < 1 || Tc > Tb) Tc = Tb;
    const int64_t nbatch = (T + Tb - 1) / Tb;
    p.bt0 = (t % nbatch) * Tb;
    p.Tn = std::min(Tb, T - p.bt0);
    // The split factor is fixed from the full chunk length; a shorter chunk re-rounds its K
    // range and can come out with more splits for the same factor, so every chunk is given the
    // effective factor of a full chunk instead: effective_splits(len, S_eff) <= S_eff.
    const int64_t S = choose_splits(m, nJ, Tc, cus);
    p.splits = effective_splits(Tc, S);
    p.gp_slices = 1;
    for (int64_t t0 = p.bt0; t0 < p.bt0 + p.Tn; t0 += Tc) {
        Chunk c;
        c.t0 = t0;
        c.len = std::min(Tc, p.bt0 + p.Tn - t0);
        c.parts_off = p.parts_total;
        // the residual launch picks its tile from (m, len), so a short chunk may switch tiles
        c.parts = clip_parts > 0 ? clip_parts : num_blocks(m, c.len, 0);
        p.parts_total += c.parts;
        p.gp_slices = std::max(p.gp_slices, effective_splits(c.len, p.splits));
        p.chunks.push_back(c);
    }
    return p;
}

std::vector<Chunk> plan_loss(int64_t m, int64_t T, int64_t Tc, int64_t* parts_total) {
    std::vector<Chunk> out;
    if (Tc < 1 || Tc > T) Tc = T;
    int64_t total = 0;
    for (int64_t t0 = 0; t0 < T; t0 += Tc) {
        Chunk c;
        c.t0 = t0;
        c.len = std::min(Tc, T - t0);
        c.parts_off = total;
        c.parts = num_blocks(m, c.len, 0);
        total += c.parts;
        out.push_back(c);
    }
    if (parts_total) *parts_total = total;
    return out;
}

}  // namespace plan
}  // namespace realq
