// CPU test of the sweep's launch planning (paper_2609_00049_amd/csrc/plan.cpp), built with
// AddressSanitizer and UndefinedBehaviorSanitizer by tests/test_host_plan.py.  It checks that the
// split-K and loss-partial workspaces a Block-GD step allocates hold everything its launches write,
// for every chunk of every step, including a short last mini-batch and a short last token chunk.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "plan.h"

using namespace realq::plan;

static int failures = 0;
#define CHECK(cond)                                                              \
    do {                                                                         \
        if (!(cond)) {                                                           \
            std::fprintf(stderr, "%s:%d: CHECK failed: %s\n", __FILE__, __LINE__, #cond); \
            ++failures;                                                          \
        }                                                                        \
    } while (0)

// Replays the writes of one planned step into buffers of exactly the planned sizes (the
// sanitizer traps any write past them): each chunk's residual launch writes one partial per block
// of its own tile choice, each gradient launch writes effective_splits(len, splits) slices.
static void replay(const StepPlan& p, int64_t m, int64_t nJ, int64_t clip_parts) {
    std::vector<double> parts((size_t)p.parts_total);
    std::vector<char> written((size_t)p.parts_total, 0);
    const int64_t slice = m * nJ;
    std::vector<float> gp((size_t)(p.gp_slices * slice));
    int64_t covered = 0;
    for (const Chunk& c : p.chunks) {
        CHECK(c.len >= 1);
        CHECK(c.t0 == p.bt0 + covered);
        covered += c.len;
        const int64_t nblk = clip_parts > 0 ? clip_parts : num_blocks(m, c.len, 0);
        CHECK(nblk == c.parts);
        for (int64_t b = 0; b < nblk; ++b) {
            parts.at((size_t)(c.parts_off + b)) = 1.0;  // at() also checks the index
            CHECK(!written[(size_t)(c.parts_off + b)]);
            written[(size_t)(c.parts_off + b)] = 1;
        }
        const int64_t z = effective_splits(c.len, p.splits);
        CHECK(z <= p.gp_slices);
        CHECK(k_per_split(c.len, p.splits) * z >= c.len);
        for (int64_t s = 0; s < z; ++s) gp[(size_t)(s * slice + slice - 1)] = 1.f;
    }
    CHECK(covered == p.Tn);
    for (char w : written) CHECK(w);  // the reduction reads every partial: each one is written
}

int main() {
    // A 512x512 layer with 8192 tokens in batches of 4160: the second batch is 4032 tokens; with
    // the full-batch split factor passed unchanged it would round to one more slice than the
    // workspace holds.
    {
        const int64_t m = 512, nJ = 384, T = 8192, Tb = 4160;
        CHECK(choose_splits(m, nJ, Tb, 256) == 16);
        CHECK(effective_splits(4160, 16) == 15 && effective_splits(4032, 16) == 16);  // the overflow
        for (int64_t t = 0; t < 4; ++t) {
            StepPlan p = plan_step(m, nJ, T, Tb, Tb, t, 256, 0);
            CHECK(p.Tn == (t % 2 == 0 ? 4160 : 4032));
            CHECK(p.splits == 15 && p.gp_slices <= p.splits);
            replay(p, m, nJ, 0);
        }
    }
    // 14336 rows, 3072 tokens in chunks of 2048: the last 1024-token chunk has fewer than 256
    // large tiles and switches to the small tile, which writes four times as many partials.
    {
        StepPlan p = plan_step(14336, 1024, 3072, 3072, 2048, 0, 256, 0);
        CHECK(p.chunks.size() == 2);
        CHECK(p.chunks[0].parts == 56 * 8);
        CHECK(p.chunks[1].parts == 112 * 8);
        CHECK(p.parts_total == 56 * 8 + 112 * 8);
        replay(p, 14336, 1024, 0);
        int64_t tot = 0;
        std::vector<Chunk> l = plan_loss(14336, 3072, 2048, &tot);
        CHECK(l.size() == 2 && tot == 56 * 8 + 112 * 8 && l[1].parts_off == 56 * 8);
    }
    // the clip writes a fixed number of partials per chunk
    {
        StepPlan p = plan_step(300, 200, 5000, 2000, 700, 2, 256, 512);
        CHECK(p.Tn == 1000);
        CHECK(p.parts_total == 2 * 512);
        replay(p, 300, 200, 512);
    }
    // the split factor of a full chunk never grows on a shorter one
    for (int64_t K = 1; K <= 9000; K += 7)
        for (int64_t s = 1; s <= 16; ++s) {
            const int64_t se = effective_splits(K, s);
            for (int64_t k2 = 1; k2 <= K; k2 += 97) CHECK(effective_splits(k2, se) <= se);
        }
    // operand rows: enough, whole 128-byte lines, an odd number of them, never shorter for more columns
    for (int64_t n = 1; n <= 20000; n += n < 300 ? 1 : 61) {
        const int64_t ld = operand_stride(n);
        CHECK(ld >= n && ld % 64 == 0 && ld / 64 % 2 == 1 && ld < n + 128);
        CHECK(operand_stride(n + 1) >= ld);
        CHECK(row_stride(n) >= n && row_stride(n) % 64 == 0 && row_stride(n) < n + 64);
    }
    // Slices of a float64-accumulated product: no float32 sum over more tokens than max_k, 256
    // tokens a slice at least otherwise, and fewer tokens never take more than 8/7 of the slices
    // that more tokens do (the room held after a larger call serves a smaller one).
    for (int64_t nt : {1, 2, 3, 5, 10, 16, 56})
        for (int64_t max_k : {0, 1024})
            for (int passes : {1, 2}) {
                int64_t most = 1;
                for (int64_t K = 1; K <= 200000; K += K < 4096 ? 5 : K < 32768 ? 64 : 1000) {
                    const int64_t q = choose_acc_splits(nt * (nt + 1) / 2, K, passes, 256, max_k);
                    CHECK(q >= 1 && q == effective_splits(K, q));
                    CHECK(max_k == 0 || k_per_split(K, q) <= max_k);
                    CHECK(q == 1 || max_k > 0 || k_per_split(K, q) >= 256);
                    CHECK(7 * most <= 8 * q);
                    most = std::max(most, q);
                }
            }
    // in one slice: straight into the matrix where the other triangle costs less than the slice
    CHECK(straight_acc(1, 16, 256) && straight_acc(4096, 1024, 256) && straight_acc(14336, 1024, 256));
    CHECK(!straight_acc(512, 16, 256) && !straight_acc(14336, 2048, 256) && !straight_acc(8192, 8192, 256));
    // Panels of such a product: whole tile rows that cover it, within the budget or one tile row
    for (int64_t M : {1, 255, 256, 257, 1000, 4097, 14336})
        for (bool sym : {false, true})
            for (int64_t slices : {1, 3, 34})
                for (int64_t budget : {int64_t(1) << 10, int64_t(100) << 20, int64_t(2) << 30}) {
                    const int64_t N = sym ? M : 1352, even = even_budget(M, N, sym, slices, budget);
                    int64_t r0 = 0, panels = 0, greedy = 0;
                    for (int64_t r = 0; r < M; ++greedy) r += panel_rows(M, N, sym, slices, r, budget);
                    CHECK(even <= budget);
                    for (; r0 < M; ++panels) {
                        const int64_t rows = panel_rows(M, N, sym, slices, r0, even);
                        CHECK(rows >= 1 && r0 + rows <= M);
                        CHECK(r0 + rows == M || rows % kLargeBM == 0);
                        CHECK(rows <= kLargeBM || panel_bytes(N, sym, slices, r0, rows) <= budget);
                        CHECK(panel_bytes(N, sym, slices, r0, rows) <=
                              std::max(budget, panel_bytes(N, false, slices, 0, std::min(M, kLargeBM))));
                        r0 += rows;
                    }
                    CHECK(panels == greedy);
                }
    // Places: every token has one of its own, in order, that leads back to it; every chunk of a step
    // is contiguous and, where tokens are apart, starts on a multiple of 8; the places without a
    // token say so and are few.
    {
        int parted = 0;
        auto check = [&](int64_t T, int64_t Tb, int64_t Tc) {
            for (bool may : {true, false}) {
                const Places L = place_tokens(T, Tb, Tc, may);
                parted += L.apart;
                CHECK(may || !L.apart);
                CHECK(L.count >= T && L.count <= T + T / 16);
                std::vector<int64_t> at((size_t)L.count, -1);
                for (int64_t t = 0; t < T; ++t) at.at((size_t)place_of(L, t)) = t;
                int64_t held = 0;
                for (int64_t p = 0; p < L.count; ++p) {
                    CHECK(token_at(L, p) == at[(size_t)p]);
                    held += at[(size_t)p] >= 0;
                }
                CHECK(held == T);
                const bool aligned = (Tb >= T || Tb % 8 == 0) && (Tc >= T || Tc % 8 == 0);
                CHECK(!(aligned && L.apart));
                for (int64_t t = 0; t < (T + Tb - 1) / Tb; ++t)
                    for (const Chunk& c : plan_step(7, 5, T, Tb, Tc, t, 256, 0).chunks) {
                        CHECK(place_of(L, c.t0 + c.len - 1) == place_of(L, c.t0) + c.len - 1);
                        CHECK(!(L.apart || aligned) || place_of(L, c.t0) % 8 == 0);
                    }
            }
        };
        for (int64_t T : {1, 7, 8, 9, 1003, 4096, 4099})
            for (int64_t Tb : {1, 8, 9, 100, 333, 336, 1001, 1002, 4099})
                for (int64_t Tc : {1, 4, 8, 63, 96, 97, 100, 101, 500, 1001, 4099}) {
                    const int64_t b = std::min(Tb, T);
                    check(T, b, std::min(Tc, b));
                }
        CHECK(parted > 20);
        CHECK(!place_tokens(262144, 9, 9).apart && place_tokens(262144, 100, 100).apart);
    }
    // randomised shapes, batches, chunks and CU counts
    std::mt19937_64 rng(1234);
    auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); };
    for (int it = 0; it < 3000; ++it) {
        const int64_t m = pick(1, 3000), nJ = pick(1, 600), T = pick(1, 20000);
        const int64_t Tb = pick(0, 1) ? T : pick(1, T);
        const int64_t Tc = pick(0, 2) == 0 ? Tb : pick(1, Tb);
        const int64_t t = pick(0, 40);
        const int cus = (int)pick(1, 304);
        const int64_t clip = pick(0, 3) == 0 ? 512 : 0;
        StepPlan p = plan_step(m, nJ, T, Tb, Tc, t, cus, clip);
        CHECK(p.Tn >= 1 && p.bt0 + p.Tn <= T);
        CHECK(p.splits >= 1 && p.splits <= 16);
        replay(p, m, nJ, clip);
    }
    if (failures) {
        std::fprintf(stderr, "%d check(s) failed\n", failures);
        return 1;
    }
    std::printf("plan: all checks passed\n");
    return 0;
}
