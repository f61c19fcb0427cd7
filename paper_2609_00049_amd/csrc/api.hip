// C ABI of the REAL-Q layer sweep (declared in include/realq.h): argument checks,
// workspace management, and the launch sequences of the five public calls.
// Everything runs on the context's stream; the only host synchronisations are the
// positive-definiteness check of realq_chol_inverse and the end of
// realq_quantize_layer.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "common.h"
#include "ctx.h"
#include "kernels.h"
#include "plan.h"
#include "../../include/realq.h"

namespace realq {

int set_error(realq_ctx* ctx, int code, const std::string& msg) {
    if (ctx) ctx->err = msg;
    return code;
}

// Frees the buffer of `slot`, if it has one, once the stream is through with it.
static int drop_ws(realq_ctx* ctx, const char* slot) {
    realq_ctx::Buf& b = ctx->ws[slot];
    if (!b.p) return REALQ_OK;
    const hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return set_error(ctx, REALQ_ERR_HIP, std::string("sync: ") + hipGetErrorString(e));
    (void)hipFree(b.p);
    b = realq_ctx::Buf();
    return REALQ_OK;
}

// Device memory for `slot` (NULL: none of the context's).  The slices of finished products are given
// back before the memory is said to be out: nothing is kept in them between calls.
static bool device_alloc(realq_ctx* ctx, const char* slot, size_t bytes, void** p) {
    for (;;) {
        if (hipMalloc(p, bytes) == hipSuccess && *p) return true;
        (void)hipGetLastError();
        *p = nullptr;
        if (!ctx->ws[kSliceSlot].p || (slot && std::strcmp(slot, kSliceSlot) == 0)) return false;
        if (drop_ws(ctx, kSliceSlot)) return false;
    }
}

int get_ws(realq_ctx* ctx, const char* slot, size_t bytes, void** out) {
    auto& b = ctx->ws[slot];
    if (bytes == 0) bytes = 16;
    if (b.bytes < bytes) {
        if (const int rc = drop_ws(ctx, slot)) return rc;
        void* p = nullptr;
        if (!device_alloc(ctx, slot, bytes, &p))
            return set_error(ctx, REALQ_ERR_OOM,
                             std::string("device allocation of ") + std::to_string(bytes) + " bytes for " + slot);
        b.p = p;
        b.bytes = bytes;
    }
    *out = b.p;
    return REALQ_OK;
}

int harvest(realq_ctx* ctx) {
    if (ctx->pending.empty()) return REALQ_OK;
    RQ_HIP(ctx, hipEventSynchronize(ctx->pending.back().b));
    for (auto& p : ctx->pending) {
        float ms = 0.f;
        RQ_HIP(ctx, hipEventElapsedTime(&ms, p.a, p.b));
        auto& s = ctx->stats[p.name];
        s.launches += 1;
        s.ms += ms;
        ctx->free_events.push_back({p.a, p.b});
    }
    ctx->pending.clear();
    return REALQ_OK;
}

}  // namespace realq

using realq::get_ws;
using realq::validate_bgd;
using realq::validate_q;
using realq::set_error;
using realq::Timed;

// ============================================================================ BGD state

struct realq_bgd_state {
    realq_ctx* ctx = nullptr;
    int64_t m = 0, n = 0, T = 0, Tc = 0;
    const float* W0 = nullptr;
    const uint16_t* X = nullptr;
    const uint16_t* Xhat = nullptr;
    const float* s = nullptr;
    const float* M = nullptr;
    const float* P = nullptr;
    realq_bgd_params prm{};
    int64_t t = 0;  // Adam step counter (one per module)
    int64_t locked = 0;  // columns [0, locked) are folded into the residual base
    bool owns = true;
    // Rows of every GEMM operand start on 16 bytes whatever n and T are (the direct-to-LDS loads need
    // it; the checked register path is about 6x slower): columns padded to ldn (plan::row_stride), tokens
    // to Tp (plan::operand_stride).  `at` gives each token's place in the token-minor arrays
    // (plan::Places).  Xg / sg are padded copies of the caller's activations and token weights in the
    // order of the places.
    int64_t ldn = 0, ldx = 0, Tp = 0;
    realq::plan::Places at;
    const uint16_t* Xg = nullptr;  // [at.count,ldx] Xhat as the GEMMs read it (ldx = n: the caller's own)
    const float* sg = nullptr;     // [at.count] token weights, or NULL
    float* B = nullptr;  // [m,Tp] residual base
    float* mA = nullptr;
    float* vA = nullptr;  // [m,n]
    uint16_t* Dhi = nullptr;
    uint16_t* Dlo = nullptr;  // [m,ldn] split(W - W0)
    uint16_t* XhT = nullptr;  // [n,Tp]
    uint16_t* Rhi = nullptr;  // split(R o s): blocked layout [m, r_ld(Tc)], or with the clip
    uint16_t* Rlo = nullptr;  // two arrays Rhi/Rlo [m, q_ld(Tc)]
    int64_t Tb = 0, nbatch = 1;  // tokens per step and number of batches (mini-batch BGD)
    float* Rf = nullptr;         // [m,q_ld(Tc)] residual kept whole for the clip
    float* tau = nullptr;        // [Tc] per-token clip thresholds
    // increments within a column block: L0 the loss of the block's first step (device scalar),
    // G0 its gradient ([m, n - c1], unscaled sum over tokens), Dacc [m,n] the weight change since
    // then and Dinc = bf16(Dacc); inc_c1 names the block they belong to (-1: none) and inc_ready
    // says Dinc holds the change of the current weights
    bool inc = false;
    double* L0 = nullptr;
    float* G0 = nullptr;
    float* Dacc = nullptr;
    uint16_t* Dinc = nullptr;
    int64_t inc_c1 = -1;
    bool inc_ready = false;
    int64_t inc_taken = 0;  // later steps taken since the block's first (at most steps - 1)
    // Gram form
    bool gram = false;
    uint16_t* Ghi = nullptr;
    uint16_t* Glo = nullptr;  // [n,ldn] split(Xhat^T S Xhat)
    float* C0 = nullptr;      // [m,n] W0 Delta^T S Xhat
    float* Pm = nullptr;      // [m,n] D Xhat^T S Xhat (per step)
    double* cconst = nullptr; // <W0 Delta^T S Delta, W0> (device scalar)
    // blended metric alpha M + (1 - alpha) P as a bf16 pair [m, row_stride(m)], formed once per alpha
    uint16_t* Mah = nullptr;
    uint16_t* Mal = nullptr;
    float Ma_alpha = -1.f;
    std::vector<void*> allocations;
};

extern "C" {

void realq_qparams_default(realq_qparams* q) {
    if (!q) return;
    q->bits = 4;
    q->group = 128;
    q->block = 128;
    q->grid = 80;
    q->damp = 0.01f;
}

void realq_bgd_params_default(realq_bgd_params* b) {
    if (!b) return;
    b->steps = 0;
    b->lr = 1e-3f;
    b->beta1 = 0.9f;
    b->beta2 = 0.999f;
    b->eps = 1e-8f;
    b->tok_chunk = 0;
    b->form = REALQ_BGD_TOKENS;
    b->loss_clip = 0.f;
    b->batch = 0;
    b->resid_increment = 1;
}

int realq_ctx_create(realq_ctx** out, void* hip_stream) {
    if (!out) return REALQ_ERR_INVALID_ARG;
    *out = nullptr;
    realq_ctx* c = new (std::nothrow) realq_ctx();
    if (!c) return REALQ_ERR_OOM;
    c->stream = (hipStream_t)hip_stream;
    if (hipGetDevice(&c->device) != hipSuccess ||
        hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) {
        (void)hipGetLastError();
        delete c;
        return REALQ_ERR_HIP;
    }
    if (c->cus < 1) c->cus = 1;
    *out = c;
    return REALQ_OK;
}

void realq_ctx_destroy(realq_ctx* ctx) {
    if (!ctx) return;
    (void)hipStreamSynchronize(ctx->stream);
    for (auto& kv : ctx->ws)
        if (kv.second.p) (void)hipFree(kv.second.p);
    for (auto& p : ctx->pending) {
        (void)hipEventDestroy(p.a);
        (void)hipEventDestroy(p.b);
    }
    for (auto& p : ctx->free_events) {
        (void)hipEventDestroy(p.first);
        (void)hipEventDestroy(p.second);
    }
    delete ctx;
}

const char* realq_last_error(const realq_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

int realq_ctx_set_timing(realq_ctx* ctx, int enable) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    ctx->timing = enable != 0;
    return REALQ_OK;
}

static const char* kTimedNames[] = {"hessian",    "chol",      "quantize",   "obs",        "lock",
                                    "resid",      "grad",      "resid_inc",  "grad_inc",   "adam",
                                    "init",       "gram",      "gram_step",  "dense_loss", "saliency",
                                    "block_init", "block_step", "attention", "metric"};

int realq_ctx_kernel_time(realq_ctx* ctx, const char* name, int64_t* launches, double* total_ms) {
    if (!ctx || !name) return REALQ_ERR_INVALID_ARG;
    bool known = false;
    for (const char* k : kTimedNames) known |= std::strcmp(k, name) == 0;
    if (!known) return set_error(ctx, REALQ_ERR_INVALID_ARG, std::string("unknown kernel name ") + name);
    int rc = realq::harvest(ctx);
    if (rc) return rc;
    auto it = ctx->stats.find(name);
    if (launches) *launches = it == ctx->stats.end() ? 0 : it->second.launches;
    if (total_ms) *total_ms = it == ctx->stats.end() ? 0.0 : it->second.ms;
    return REALQ_OK;
}

int realq_ctx_reset_timing(realq_ctx* ctx) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    int rc = realq::harvest(ctx);
    ctx->stats.clear();
    return rc;
}

// ============================================================================ a1: Hessian

}  // extern "C"

// Tokens per chunk of the products over tokens (about 256 MB of a transposed chunk), and the bytes
// of one such chunk.
static int64_t token_chunk(int64_t n, int64_t T) {
    const int64_t tc = ((int64_t)128 << 20) / n;
    return std::min(tc < 256 ? 256 : tc / 256 * 256, (T + 7) / 8 * 8);
}
static int64_t gram_staging(int64_t n, int64_t T) { return n * realq::plan::operand_stride(token_chunk(n, T)) * 2; }

static hipError_t acc_direct(const realq::GemmArgs& g, double* C, int64_t ldc, bool, hipStream_t st) {
    return realq::gemm_acc_f64(g, C, ldc, st);
}
static hipError_t acc_direct(const realq::GemmArgs& g, float* C, int64_t ldc, bool store, hipStream_t st) {
    return store ? realq::gemm_store_f32(g, C, ldc, 0, 1.f, st) : realq::gemm_acc_f32(g, C, ldc, 1.f, st);
}

// Most bytes the slices of sum_products hold; larger products are formed in panels of rows.
static constexpr int64_t kSliceBytes = (int64_t)3 << 30;

// Whether the stream records a graph: no memory can be allocated then.
static bool capturing(realq_ctx* ctx) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(ctx->stream, &st) != hipSuccess) (void)hipGetLastError();
    return st != hipStreamCaptureStatusNone;
}

// Room for product slices: `want` bytes, or what the context holds when that is at least 7/8 of it
// (fewer tokens can take up to 1.13 times the slices) or the stream records a graph (fewer columns can
// take more of them too), or as much as there is, down to `least`; 0 when there is not that.
static int64_t slice_room(realq_ctx* ctx, int64_t want, int64_t least, void** S, int* rc) {
    const int64_t held = (int64_t)ctx->ws[realq::kSliceSlot].bytes;
    if (held < want && capturing(ctx)) {
        if (held < least) {
            *rc = REALQ_ERR_OOM;
            return 0;
        }
        want = held;
    }
    if (held >= least && held >= want / 8 * 7) want = held;
    for (;; want = std::max(least, want / 2)) {
        *rc = get_ws(ctx, realq::kSliceSlot, (size_t)want, S);
        if (*rc == REALQ_OK) return want;
        if (*rc != REALQ_ERR_OOM || want == least) return 0;
    }
}

// C (+)= the sum of count products A_p B_p^T (M x N, g[p].K wide each, Alo optional) in float64:
// each product in float32 slices over ranges of K (split-K fills the chip whatever M and N are; a
// slice's float32 sums are shorter), the slices summed into C in float64 in a fixed order.
// symmetric: the sum of products is a symmetric matrix; only its lower tiles are formed.  flag
// (device, may be NULL): the products from `always` on are only formed when it reads nonzero.
// max_k > 0 bounds the terms of a float32 sum of the hi/lo products (with weights of several orders
// of magnitude a few tokens carry H, and what later tokens' additions to them round away shows in
// the last codes of a sweep: 1024 tokens a sum leave 2e-7 of H where 8192 left 6e-7).
// The slices are held for one panel of rows at a time; how many panels changes no sum.
template <class Out>
static int sum_products(realq_ctx* ctx, realq::GemmArgs* g, int count, int always, const int* flag, bool symmetric,
                        int64_t max_k, bool accumulate, Out* C, int64_t ldc) {
    const int64_t M = g[0].M, N = g[0].N;
    const int64_t nt = (M + realq::plan::kLargeBM - 1) / realq::plan::kLargeBM;
    const int64_t tiles = symmetric ? nt * (nt + 1) / 2 : realq::plan::tiles(M, N, true);
    hipStream_t s = ctx->stream;
    int64_t total = 0, first = 0;
    for (int p = 0; p < count; ++p) {
        g[p].run_if = p >= always ? flag : nullptr;
        g[p].splits = realq::plan::choose_acc_splits(tiles, g[p].K, g[p].Alo ? 2 : 1, ctx->cus, g[p].Alo ? max_k : 0);
        total += realq::gemm_effective_splits(g[p].K, g[p].splits);
        if (p + 1 == always) first = total;
    }
    // a single slice holds the very sums that go into C; the terms of a weighted symmetric product do
    // not make a symmetric matrix by themselves
    if (total == 1 && accumulate && (!symmetric || (!g[0].Alo && realq::plan::straight_acc(M, g[0].K, ctx->cus)))) {
        RQ_HIP(ctx, acc_direct(g[0], C, ldc, false, s));
        return REALQ_OK;
    }
    // one row of tiles over all columns; never more than the whole
    const int64_t least = realq::plan::panel_bytes(N, false, total, 0, std::min(M, realq::plan::kLargeBM));
    const int64_t all = realq::plan::panel_bytes(N, symmetric, total, 0, M);
    void* S;
    int rc;
    const int64_t room = slice_room(ctx, std::max(least, std::min(all, kSliceBytes)), least, &S, &rc);
    if (rc == REALQ_ERR_OOM) {  // not even one row of tiles: straight into C, both triangles
        for (int p = 0; p < count; ++p) {
            const int64_t step = g[p].Alo && max_k > 0 ? max_k : g[p].K;
            for (int64_t k0 = 0; k0 < g[p].K; k0 += step) {
                realq::GemmArgs q = g[p];
                q.Ahi += k0;
                if (q.Alo) q.Alo += k0;
                q.B += k0;
                q.K = std::min(step, g[p].K - k0);
                q.splits = 1;
                RQ_HIP(ctx, acc_direct(q, C, ldc, p == 0 && k0 == 0 && !accumulate, s));
            }
        }
        return REALQ_OK;
    }
    if (rc) return rc;
    const int64_t budget = realq::plan::even_budget(M, N, symmetric, total, room);
    for (int64_t r0 = 0; r0 < M;) {
        const int64_t rows = realq::plan::panel_rows(M, N, symmetric, total, r0, budget);
        const int64_t cols = symmetric ? r0 + rows : N;
        float* out = (float*)S;
        for (int p = 0; p < count; ++p) {
            realq::GemmArgs q = g[p];
            q.Ahi += r0 * q.lda;
            if (q.Alo) q.Alo += r0 * q.lda;
            q.M = rows;
            q.N = symmetric ? r0 : N;  // symmetric: the columns left of the panel's own square, if any
            RQ_HIP(ctx, realq::gemm_grad(q, out, cols, rows * cols, s));
            if (symmetric) {
                q.B += r0 * q.ldb;
                q.N = rows;
                q.tri = 1;
                RQ_HIP(ctx, realq::gemm_grad(q, out + r0, cols, rows * cols, s));
            }
            out += realq::gemm_effective_splits(q.K, q.splits) * rows * cols;
        }
        RQ_HIP(ctx, realq::add_slices((const float*)S, first, total, flag, r0, r0 + rows, N, symmetric, accumulate, C,
                                      ldc, s));
        r0 += rows;
    }
    return REALQ_OK;
}

// Token chunks of tc tokens staged in caller-provided bf16 buffers of n rows of ld >= tc elements each
// (xt, and hi, lo, lo2 when s is given): the chunk transposed (and, with weights, s_t xhat_t split into three
// bf16 terms), then H_acc += chunk^T chunk on MFMA.  alloc = false (the allocation-free entry point)
// adds the products straight into H_acc and skips the timing events.
int realq::hessian_accum_chunks(realq_ctx* ctx, const uint16_t* Xhat, const float* s, int64_t T, int64_t n,
                                double* H_acc, int64_t tc, int64_t ld, uint16_t* xt, uint16_t* hi, uint16_t* lo,
                                uint16_t* lo2, bool alloc) {
    Timed tm(ctx, alloc ? "hessian" : nullptr);
    for (int64_t t0 = 0; t0 < T; t0 += tc) {
        const int64_t cur = std::min(tc, T - t0);
        // s_t xhat_t in three bf16 terms: with a heavy-tailed s a few tokens carry H, and the
        // 2^-17 remainder of a hi/lo pair would not average out over the tokens
        if (s)
            RQ_HIP(ctx, realq::transpose_scale_split(Xhat + t0 * n, n, s + t0, xt, hi, lo, lo2, ld, cur, n, ctx->stream));
        else
            RQ_HIP(ctx, realq::transpose_u16(Xhat + t0 * n, n, xt, ld, cur, n, ctx->stream));
        realq::GemmArgs g[2] = {{s ? hi : xt, s ? lo : nullptr, ld, xt, ld, n, n, cur, 1},
                                {lo2, nullptr, ld, xt, ld, n, n, cur, 1}};
        const int count = s ? 2 : 1;
        if (alloc) {
            const int rc = sum_products(ctx, g, count, count, nullptr, true, s ? 1024 : 0, true, H_acc, n);
            if (rc) return rc;
        } else {
            for (int p = 0; p < count; ++p) RQ_HIP(ctx, realq::gemm_acc_f64(g[p], H_acc, n, ctx->stream));
        }
    }
    return REALQ_OK;
}

extern "C" {

int realq_hessian_accum(realq_ctx* ctx, const uint16_t* Xhat, const float* s, int64_t T, int64_t n, double* H_acc) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    if (T < 0 || n <= 0) return set_error(ctx, REALQ_ERR_SHAPE, "hessian_accum: need T >= 0, n > 0");
    if (T == 0) return REALQ_OK;
    if (!Xhat || !H_acc) return set_error(ctx, REALQ_ERR_INVALID_ARG, "hessian_accum: NULL Xhat or H_acc");
    // token chunk bounded so the transposed workspace stays near 256 MiB per operand
    const int64_t tc = token_chunk(n, T), ld = realq::plan::operand_stride(tc);
    void *xt = nullptr, *hi = nullptr, *lo = nullptr, *lo2 = nullptr;
    int rc = get_ws(ctx, "h_xt", (size_t)n * ld * 2, &xt);
    if (rc) return rc;
    if (s) {
        if ((rc = get_ws(ctx, "h_hi", (size_t)n * ld * 2, &hi))) return rc;
        if ((rc = get_ws(ctx, "h_lo", (size_t)n * ld * 2, &lo))) return rc;
        if ((rc = get_ws(ctx, "h_lo2", (size_t)n * ld * 2, &lo2))) return rc;
    }
    return realq::hessian_accum_chunks(ctx, Xhat, s, T, n, H_acc, tc, ld, (uint16_t*)xt, (uint16_t*)hi, (uint16_t*)lo,
                                       (uint16_t*)lo2, true);
}

// ============================================================================ a0: Stage-0 accumulators

int realq_fisher_accum(realq_ctx* ctx, const uint16_t* G, int64_t T, int64_t m, double* F_acc) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    if (T < 0 || m <= 0) return set_error(ctx, REALQ_ERR_SHAPE, "fisher_accum: need T >= 0, m > 0");
    if (T == 0) return REALQ_OK;
    if (!G || !F_acc) return set_error(ctx, REALQ_ERR_INVALID_ARG, "fisher_accum: NULL G or F_acc");
    // sum_t g_t g_t^T is the unweighted Hessian contraction with the gradients in place of the inputs
    return realq_hessian_accum(ctx, G, nullptr, T, m, F_acc);
}

int realq_fisher_finish(realq_ctx* ctx, const double* F_acc, int64_t m, int64_t T_total, float* F) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    if (m <= 0 || T_total <= 0) return set_error(ctx, REALQ_ERR_SHAPE, "fisher_finish: need m > 0, T_total > 0");
    if (!F_acc || !F) return set_error(ctx, REALQ_ERR_INVALID_ARG, "fisher_finish: NULL F_acc or F");
    RQ_HIP(ctx, realq::div_narrow(F_acc, (double)T_total, F, m * m, ctx->stream));
    return REALQ_OK;
}

int realq_saliency(realq_ctx* ctx, const uint16_t* G, int64_t T, int64_t m, int32_t n_groups, float clip_q,
                   float* s_out) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    if (T < 0 || m <= 0) return set_error(ctx, REALQ_ERR_SHAPE, "saliency: need T >= 0, m > 0");
    if (n_groups < 1 || n_groups > m) return set_error(ctx, REALQ_ERR_INVALID_ARG, "saliency: need 1 <= n_groups <= m");
    if (!std::isfinite(clip_q) || clip_q < 0.f || clip_q > 1.f)
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "saliency: clip_q must lie in [0, 1] (0 = off)");
    if (T == 0) return REALQ_OK;
    if (!G || !s_out) return set_error(ctx, REALQ_ERR_INVALID_ARG, "saliency: NULL G or s_out");
    const int64_t k = clip_q > 0.f ? std::max<int64_t>(1, (int64_t)std::ceil((double)clip_q * (double)T)) : 0;
    void *s64, *tau, *sel;
    int rc;
    if ((rc = get_ws(ctx, "sal_s", (size_t)n_groups * T * 8, &s64))) return rc;
    if ((rc = get_ws(ctx, "sal_tau", (size_t)n_groups * 8, &tau))) return rc;
    if ((rc = get_ws(ctx, "sal_sel", (size_t)realq::saliency_select_bytes(n_groups), &sel))) return rc;
    Timed tm(ctx, "saliency");
    RQ_HIP(ctx, realq::saliency(G, T, m, n_groups, k, (double*)s64, (double*)tau, sel, s_out, ctx->stream));
    return REALQ_OK;
}

// ============================================================================ a2: inverse factor

int realq_chol_inverse(realq_ctx* ctx, const double* H_acc, int64_t n, int64_t T_total, float damp, float* H_out,
                       float* U, uint8_t* dead) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    if (n <= 0 || T_total <= 0) return set_error(ctx, REALQ_ERR_SHAPE, "chol_inverse: need n > 0 and T_total > 0");
    if (!H_acc || !U) return set_error(ctx, REALQ_ERR_INVALID_ARG, "chol_inverse: NULL H_acc or U");
    if (!(damp > 0.f) || !std::isfinite(damp))
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "chol_inverse: damp must be finite and > 0");
    const int64_t np = ((n + 63) / 64) * 64;
    void *A, *L, *F, *S;
    int rc;
    if ((rc = get_ws(ctx, "c_A", (size_t)np * np * 8, &A))) return rc;
    if ((rc = get_ws(ctx, "c_L", (size_t)np * np * 8, &L))) return rc;
    if ((rc = get_ws(ctx, "c_F", 64, &F))) return rc;
    if ((rc = get_ws(ctx, "c_S", 64, &S))) return rc;
    // two flag words (not positive definite; non-finite accumulator) cleared by one double fill
    RQ_HIP(ctx, realq::fill_f64((double*)F, 0.0, 1, ctx->stream));
    realq::CholArgs c{};
    c.Hacc = H_acc;
    c.n = n;
    c.np = np;
    c.scale = 2.0 / (double)T_total;
    c.damp = damp;
    c.Hout = H_out;
    c.dead = dead;
    c.A = (double*)A;
    c.Linv = (double*)L;
    c.flag = (int*)F;
    c.scratch = (double*)S;
    c.U = U;
    {
        Timed tm(ctx, "chol");
        RQ_HIP(ctx, realq::chol_inverse(c, ctx->stream));
    }
    int flag[2] = {0, 0};
    RQ_HIP(ctx, hipMemcpyAsync(flag, F, sizeof(flag), hipMemcpyDeviceToHost, ctx->stream));
    RQ_HIP(ctx, hipStreamSynchronize(ctx->stream));
    if (flag[1])
        return set_error(ctx, REALQ_ERR_NONFINITE,
                         "chol_inverse: the Hessian accumulator holds NaN or Inf (non-finite Xhat or s)");
    if (flag[0]) return set_error(ctx, REALQ_ERR_NOT_SPD, "chol_inverse: damped Hessian is not positive definite");
    return REALQ_OK;
}

// ============================================================================ BGD state

// Row stride (bf16 values) of split(R o s) in the blocked layout for `cur` tokens: hi and lo of
// every 32 tokens, rounded up to an operand stride.
static int64_t r_ld(int64_t cur) { return realq::plan::operand_stride(2 * ((cur + 31) / 32) * 32); }
// row stride of bf16(acc o s) on a later step of a column block (row-major, in the same buffer)
static int64_t q_ld(int64_t cur) { return realq::plan::operand_stride(cur); }

static int state_alloc(realq_bgd_state* st, void** p, size_t bytes, const char* slot) {
    realq_ctx* ctx = st->ctx;
    if (!st->owns) return get_ws(ctx, slot, bytes, p);
    *p = nullptr;
    if (!realq::device_alloc(ctx, nullptr, bytes ? bytes : 16, p))
        return set_error(ctx, REALQ_ERR_OOM, std::string("device allocation of ") + std::to_string(bytes) + " bytes");
    st->allocations.push_back(*p);
    return REALQ_OK;
}

static void state_free(realq_bgd_state* st) {
    if (!st) return;
    if (st->ctx) (void)hipStreamSynchronize(st->ctx->stream);
    for (void* p : st->allocations) (void)hipFree(p);
    st->allocations.clear();
}

// Calibration Gram matrices of the input perturbation Delta = Xhat - X, accumulated over token
// chunks in float64: Gdh = Delta^T S Xhat and Gdd = Delta^T S Delta (S = diag(s) or I).  The
// float32 operand s o Delta is carried as a hi/lo bf16 pair against Xhat (bf16) and against
// both halves of Delta.
static int gram_accum(realq_ctx* ctx, const uint16_t* Xhat, const uint16_t* X, const float* sw, int64_t T, int64_t n,
                      double* Gdh, double* Gdd) {
    hipStream_t s = ctx->stream;
    int rc;
    void *sdh, *sdl, *dh, *dl, *xt;
    const int64_t tc = token_chunk(n, T), ld = realq::plan::operand_stride(tc);
    const size_t staging = (size_t)gram_staging(n, T);
    if ((rc = get_ws(ctx, "g_sdh", staging, &sdh))) return rc;
    if ((rc = get_ws(ctx, "g_sdl", staging, &sdl))) return rc;
    if ((rc = get_ws(ctx, "g_dh16", staging, &dh))) return rc;
    if ((rc = get_ws(ctx, "g_dl16", staging, &dl))) return rc;
    if ((rc = get_ws(ctx, "g_xt", staging, &xt))) return rc;
    Timed tm(ctx, "gram");
    RQ_HIP(ctx, realq::fill_f64(Gdh, 0.0, n * n, s));
    RQ_HIP(ctx, realq::fill_f64(Gdd, 0.0, n * n, s));
    for (int64_t t0 = 0; t0 < T; t0 += tc) {
        const int64_t cur = std::min(tc, T - t0);
        RQ_HIP(ctx, realq::transpose_delta_split(Xhat + t0 * n, X + t0 * n, n, sw ? sw + t0 : nullptr, (uint16_t*)sdh,
                                                 (uint16_t*)sdl, (uint16_t*)dh, (uint16_t*)dl, ld, cur, n, s));
        RQ_HIP(ctx, realq::transpose_u16(Xhat + t0 * n, n, (uint16_t*)xt, ld, cur, n, s));
        realq::GemmArgs g{(const uint16_t*)sdh, (const uint16_t*)sdl, ld, (const uint16_t*)xt, ld, n, n, cur, 1};
        if ((rc = sum_products(ctx, &g, 1, 1, nullptr, false, 0, true, Gdh, n))) return rc;
        realq::GemmArgs gd[2] = {g, g};
        gd[0].B = (const uint16_t*)dh;
        gd[1].B = (const uint16_t*)dl;
        if ((rc = sum_products(ctx, gd, 2, 2, nullptr, true, 0, true, Gdd, n))) return rc;
    }
    return REALQ_OK;
}

extern "C++" {
int realq::validate_bgd(realq_ctx* ctx, const realq_bgd_params* p) {
    if (!p) return set_error(ctx, REALQ_ERR_INVALID_ARG, "NULL bgd params");
    if (p->steps < 0) return set_error(ctx, REALQ_ERR_INVALID_ARG, "bgd steps must be >= 0");
    if (!std::isfinite(p->lr) || p->lr < 0.f) return set_error(ctx, REALQ_ERR_INVALID_ARG, "lr must be finite, >= 0");
    if (!(p->beta1 >= 0.f && p->beta1 < 1.f) || !(p->beta2 >= 0.f && p->beta2 < 1.f))
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "Adam betas must lie in [0, 1)");
    if (!(p->eps > 0.f)) return set_error(ctx, REALQ_ERR_INVALID_ARG, "Adam eps must be > 0");
    if (p->tok_chunk < 0) return set_error(ctx, REALQ_ERR_INVALID_ARG, "tok_chunk must be >= 0");
    if (p->form != REALQ_BGD_TOKENS && p->form != REALQ_BGD_GRAM)
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "form must be REALQ_BGD_TOKENS or REALQ_BGD_GRAM");
    if (!std::isfinite(p->loss_clip) || p->loss_clip < 0.f || p->loss_clip > 1.f)
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "loss_clip must lie in [0, 1] (0 = off)");
    if (p->batch < 0) return set_error(ctx, REALQ_ERR_INVALID_ARG, "batch must be >= 0");
    if (p->resid_increment != 0 && p->resid_increment != 1)
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "resid_increment must be 0 or 1");
    return REALQ_OK;
}
}  // extern "C++"

static int state_init_gram(realq_bgd_state* st);

// Whether steps after a block's first may take residual and gradient as increments
// (resid_increment in realq.h).  Adam's step is at most lr (1 - b1) / sqrt((1 - b2)(1 - b1^2/b2))
// for any gradient history (Cauchy-Schwarz on the two moment sums, bias corrections included), so
// the weight change over the steps - 1 later steps of a block is at most that times steps - 1;
// the increments are taken when this bound is within rms(W0) / 32, the module has at most
// kIncMaxColumns input columns (64 column blocks) and at least kIncTokensPerColumn tokens per
// input column.
static constexpr int64_t kIncMaxColumns = 8192;
static constexpr int64_t kIncTokensPerColumn = 16;
static int inc_init(realq_bgd_state* st) {
    realq_ctx* ctx = st->ctx;
    const realq_bgd_params& p = st->prm;
    st->inc = false;
    st->inc_c1 = -1;
    st->inc_ready = false;
    const double b1 = p.beta1, b2 = p.beta2;
    const int64_t m = st->m, n = st->n, T = st->T;
    if (!p.resid_increment || p.steps < 2 || p.loss_clip > 0.f || st->Tb != T || !(b1 * b1 < b2) ||
        n > kIncMaxColumns || T < kIncTokensPerColumn * n)
        return REALQ_OK;
    const double step_max = (1.0 - b1) / std::sqrt((1.0 - b2) * (1.0 - b1 * b1 / b2));
    const double disp = (double)(p.steps - 1) * step_max * (double)p.lr;
    void *parts, *ms;
    int rc;
    if ((rc = get_ws(ctx, "i_parts", (size_t)realq::dot_f32_partials() * 8, &parts))) return rc;
    if ((rc = get_ws(ctx, "i_ms", 8, &ms))) return rc;
    RQ_HIP(ctx, realq::dot_f32(st->W0, st->W0, m * n, 1.0, (double*)parts, ctx->stream));
    RQ_HIP(ctx, realq::reduce_partials((const double*)parts, realq::dot_f32_partials(), 1.0 / ((double)m * (double)n),
                                       (double*)ms, ctx->stream));
    double msq = 0.0;
    RQ_HIP(ctx, hipMemcpyAsync(&msq, ms, 8, hipMemcpyDeviceToHost, ctx->stream));
    RQ_HIP(ctx, hipStreamSynchronize(ctx->stream));
    if (!(disp <= std::sqrt(msq) / 32.0)) return REALQ_OK;
    void* q;
    if ((rc = state_alloc(st, &q, 8, "s_L0"))) return rc;
    st->L0 = (double*)q;
    if ((rc = state_alloc(st, &q, (size_t)m * n * 4, "s_Dacc"))) return rc;
    st->Dacc = (float*)q;
    if ((rc = state_alloc(st, &q, (size_t)m * st->ldn * 2, "s_Dinc"))) return rc;
    st->Dinc = (uint16_t*)q;
    if ((rc = state_alloc(st, &q, (size_t)m * n * 4, "s_G0"))) return rc;
    st->G0 = (float*)q;
    st->inc = true;
    return REALQ_OK;
}

// A device buffer: its slot among the context workspaces, its size and, for the arrays of a state,
// where its address goes.
struct Array {
    const char* slot;
    int64_t bytes;
    void (*put)(realq_bgd_state*, void*);
};

// The arrays of a token-form state (sizes from its tokens' places).
static std::vector<Array> state_arrays(const realq_bgd_state* st) {
    using S = realq_bgd_state;
    const int64_t m = st->m, n = st->n, Tc = st->Tc, ldn = st->ldn, Tp = st->Tp;
    const bool clip = st->prm.loss_clip > 0.f;
    std::vector<Array> v{{"s_B", m * Tp * 4, [](S* s, void* p) { s->B = (float*)p; }},
                         {"s_m", m * n * 4, [](S* s, void* p) { s->mA = (float*)p; }},
                         {"s_v", m * n * 4, [](S* s, void* p) { s->vA = (float*)p; }},
                         {"s_Dh", m * ldn * 2, [](S* s, void* p) { s->Dhi = (uint16_t*)p; }},
                         {"s_Dl", m * ldn * 2, [](S* s, void* p) { s->Dlo = (uint16_t*)p; }},
                         {"s_XT", n * Tp * 2, [](S* s, void* p) { s->XhT = (uint16_t*)p; }},
                         // with the clip split(R o s) as two arrays, else one of 128-byte lines (32 tokens'
                         // hi, then their lo): whole-line stores
                         {"s_Rh", m * (clip ? q_ld(Tc) : r_ld(Tc)) * 2, [](S* s, void* p) { s->Rhi = (uint16_t*)p; }}};
    if (clip) {
        v.push_back({"s_Rl", m * q_ld(Tc) * 2, [](S* s, void* p) { s->Rlo = (uint16_t*)p; }});
        v.push_back({"s_Rf", m * q_ld(Tc) * 4, [](S* s, void* p) { s->Rf = (float*)p; }});
        v.push_back({"s_tau", Tc * 4, [](S* s, void* p) { s->tau = (float*)p; }});
    }
    if (st->s && st->at.apart) v.push_back({"s_sg", st->at.count * 4, [](S* s, void* p) { s->sg = (float*)p; }});
    return v;
}

// Whether a copy of the activations in `bytes` leaves room for what a sweep allocates after it: the
// state's arrays, the workspaces of its steps and of the final loss (at their largest), 64 MB for
// the small ones.  The copy only makes products faster; those it cannot do without.
static bool copy_fits(realq_bgd_state* st, int64_t bytes) {
    realq_ctx* ctx = st->ctx;
    const int64_t m = st->m, n = st->n, mp = realq::plan::row_stride(m), ldn = st->ldn;
    const bool dense = st->M || st->P;
    std::vector<Array> v = state_arrays(st);
    v.push_back({"s_Xg", bytes, nullptr});
    int64_t gp = 0;
    for (int64_t nJ = n; nJ > 0; nJ -= 128)  // the split factor falls with the columns, not evenly
        gp = std::max(gp, realq::plan::choose_splits(m, nJ, st->Tc, ctx->cus) * m * nJ * 4);
    v.insert(v.end(), {{"b_Gp", gp, nullptr}, {"b_G", m * n * 4, nullptr}, {"q_E", m * 128 * 8, nullptr},
                       {"l_W", m * n * 8, nullptr}});
    const int64_t chunk = std::min(st->at.count * ldn * 2, (int64_t)256 << 20);
    if (st->X != st->Xhat) v.insert(v.end(), {{"i_xh", chunk, nullptr}, {"i_xl", chunk, nullptr}});
    if (st->prm.resid_increment && st->prm.steps > 1)
        v.insert(v.end(), {{"s_Dacc", m * n * 4, nullptr}, {"s_Dinc", m * ldn * 2, nullptr},
                           {"s_G0", m * n * 4, nullptr}});
    if (dense)
        v.insert(v.end(), {{"s_Mah", m * mp * 2, nullptr}, {"s_Mal", m * mp * 2, nullptr}, {"b_Gm", m * n * 4, nullptr},
                           {"b_GTh", mp * n * 2, nullptr}, {"b_GTl", mp * n * 2, nullptr}});
    if (st->M) {
        for (const char* slot : {"g_sdh", "g_sdl", "g_dh16", "g_dl16", "g_xt"})
            v.push_back({slot, gram_staging(n, st->T), nullptr});
        for (const char* slot : {"g_A", "g_D", "g_E", "g_MX"}) v.push_back({slot, m * n * 8, nullptr});
        v.insert(v.end(), {{"g_dh", n * n * 8, nullptr}, {"g_dd", n * n * 8, nullptr}, {"g_M", m * m * 8, nullptr}});
    }
    int64_t need = 0;
    for (const Array& a : v) {  // a buffer that the context holds grows
        auto it = ctx->ws.find(a.slot);
        const bool own = st->owns && a.slot[0] == 's';
        need += std::max<int64_t>(0, a.bytes - (own || it == ctx->ws.end() ? 0 : (int64_t)it->second.bytes));
    }
    if (need == 0) return true;
    need += (int64_t)64 << 20;
    size_t free_bytes = 0, total = 0;
    if (hipMemGetInfo(&free_bytes, &total) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return need <= (int64_t)free_bytes + (int64_t)ctx->ws[realq::kSliceSlot].bytes;
}

static int state_init(realq_bgd_state* st) {
    if (st->prm.form == REALQ_BGD_GRAM) return state_init_gram(st);
    realq_ctx* ctx = st->ctx;
    const int64_t m = st->m, n = st->n, T = st->T;
    hipStream_t s = ctx->stream;
    st->gram = false;
    st->Tb = (st->prm.batch > 0 && st->prm.batch < T) ? st->prm.batch : T;
    st->nbatch = (T + st->Tb - 1) / st->Tb;
    const int64_t Tc = st->Tc = st->prm.tok_chunk > 0 ? std::min<int64_t>(st->prm.tok_chunk, st->Tb) : st->Tb;
    const int64_t ldn = st->ldn = realq::plan::row_stride(n);
    int rc;
    void* p;
    auto place = [&](bool may_part) {
        st->at = realq::plan::place_tokens(T, st->Tb, Tc, may_part);
        st->Tp = realq::plan::operand_stride(st->at.count);
    };
    place(true);
    // The activations are copied where their rows or places differ from the caller's.  The copy costs one
    // read and write of Xhat against a residual product per Block-GD step; without steps aligned
    // rows stay where they are, and without room for it all rows do, with the tokens in their order.
    st->Xg = st->Xhat;
    st->ldx = n;
    if (st->at.apart || (ldn != n && (n % 8 || st->prm.steps > 0))) {
        const int64_t bytes = st->at.count * ldn * 2;
        rc = copy_fits(st, bytes) ? state_alloc(st, &p, (size_t)bytes, "s_Xg") : REALQ_ERR_OOM;
        if (rc && rc != REALQ_ERR_OOM) return rc;
        if (rc) {
            place(false);
            if (!st->owns && (rc = realq::drop_ws(ctx, "s_Xg"))) return rc;
        } else {
            st->Xg = (const uint16_t*)p;
            st->ldx = ldn;
        }
    }
    st->sg = st->s;
    for (const Array& a : state_arrays(st)) {
        if ((rc = state_alloc(st, &p, (size_t)a.bytes, a.slot))) return rc;
        a.put(st, p);
    }
    const realq::plan::Places& at = st->at;
    const int64_t Tp = st->Tp;

    Timed tm(ctx, "init");
    RQ_HIP(ctx, realq::fill_f32(st->mA, 0.f, m * n, s));
    RQ_HIP(ctx, realq::fill_f32(st->vA, 0.f, m * n, s));
    if (st->Xg != st->Xhat)
        RQ_HIP(ctx, realq::place_rows_u16(st->Xhat, n, const_cast<uint16_t*>(st->Xg), ldn, n, at, s));
    if (st->sg != st->s) RQ_HIP(ctx, realq::place_f32(st->s, const_cast<float*>(st->sg), at, s));
    RQ_HIP(ctx, realq::transpose_u16(st->Xg, st->ldx, st->XhT, Tp, at.count, n, s));
    // Residual base before any block is locked: B = W0 (Xhat - X)^T.
    if (st->X == st->Xhat) {
        RQ_HIP(ctx, realq::fill_f32(st->B, 0.f, m * Tp, s));
    } else {
        // W0 = W0hi + W0lo (in the D buffers for now), Xhat - X = Dxh + Dxl (bf16 pairs, exact
        // difference in float32 first): B = W0 Dxh^T (both halves of W0) + W0hi Dxl^T.
        RQ_HIP(ctx, realq::split_diff_f32(st->W0, n, nullptr, 0, st->Dhi, st->Dlo, ldn, m, n, s));
        const int64_t tcx = std::max<int64_t>(8, std::min(at.count, ((int64_t)(256ll << 20) / (2 * ldn) / 8) * 8));
        void *xh, *xl;
        if ((rc = get_ws(ctx, "i_xh", (size_t)tcx * ldn * 2, &xh))) return rc;
        if ((rc = get_ws(ctx, "i_xl", (size_t)tcx * ldn * 2, &xl))) return rc;
        for (int64_t p0 = 0; p0 < at.count; p0 += tcx) {
            const int64_t cur = std::min(tcx, at.count - p0);
            RQ_HIP(ctx, realq::split_diff_bf16(st->Xhat, st->X, (uint16_t*)xh, (uint16_t*)xl, ldn, cur, n, at, p0, s));
            realq::GemmArgs g{st->Dhi, st->Dlo, ldn, (const uint16_t*)xh, ldn, m, cur, n, 1};
            RQ_HIP(ctx, realq::gemm_store_f32(g, st->B + p0, Tp, 0, 1.f, s));
            realq::GemmArgs g2{st->Dhi, nullptr, ldn, (const uint16_t*)xl, ldn, m, cur, n, 1};
            RQ_HIP(ctx, realq::gemm_acc_f32(g2, st->B + p0, Tp, 1.f, s));
        }
    }
    RQ_HIP(ctx, realq::fill_u16(st->Dhi, 0, m * ldn, s));
    RQ_HIP(ctx, realq::fill_u16(st->Dlo, 0, m * ldn, s));
    st->t = 0;
    st->locked = 0;
    return inc_init(st);
}

// Gram form: the three calibration Gram matrices once, then C0 = W0 G_dh and the constant
// c = <W0 G_dd, W0>; no residual base and no transposed activations are kept.
static int state_init_gram(realq_bgd_state* st) {
    realq_ctx* ctx = st->ctx;
    const int64_t m = st->m, n = st->n, T = st->T;
    hipStream_t s = ctx->stream;
    st->gram = true;
    st->Tc = T;
    st->Tb = T;
    st->nbatch = 1;
    const int64_t ldn = st->ldn = realq::plan::row_stride(n);
    int rc;
    void* p;
    if ((rc = state_alloc(st, &p, (size_t)m * n * 4, "s_m"))) return rc;
    st->mA = (float*)p;
    if ((rc = state_alloc(st, &p, (size_t)m * n * 4, "s_v"))) return rc;
    st->vA = (float*)p;
    if ((rc = state_alloc(st, &p, (size_t)m * ldn * 2, "s_Dh"))) return rc;
    st->Dhi = (uint16_t*)p;
    if ((rc = state_alloc(st, &p, (size_t)m * ldn * 2, "s_Dl"))) return rc;
    st->Dlo = (uint16_t*)p;
    if ((rc = state_alloc(st, &p, (size_t)n * ldn * 2, "s_Gh"))) return rc;
    st->Ghi = (uint16_t*)p;
    if ((rc = state_alloc(st, &p, (size_t)n * ldn * 2, "s_Gl"))) return rc;
    st->Glo = (uint16_t*)p;
    if ((rc = state_alloc(st, &p, (size_t)m * n * 4, "s_C0"))) return rc;
    st->C0 = (float*)p;
    if ((rc = state_alloc(st, &p, (size_t)m * n * 4, "s_P"))) return rc;
    st->Pm = (float*)p;
    if ((rc = state_alloc(st, &p, 8, "s_c"))) return rc;
    st->cconst = (double*)p;
    void *ghh, *gdh, *gdd, *A, *E, *parts;
    const int64_t np = realq::dot_f64_partials();
    if ((rc = get_ws(ctx, "i_Ghh", (size_t)n * n * 8, &ghh))) return rc;
    if ((rc = get_ws(ctx, "i_Gdh", (size_t)n * n * 8, &gdh))) return rc;
    if ((rc = get_ws(ctx, "i_Gdd", (size_t)n * n * 8, &gdd))) return rc;
    if ((rc = get_ws(ctx, "i_A", (size_t)m * n * 8, &A))) return rc;
    if ((rc = get_ws(ctx, "i_E", (size_t)m * n * 8, &E))) return rc;
    if ((rc = get_ws(ctx, "i_parts", (size_t)np * 8, &parts))) return rc;
    RQ_HIP(ctx, realq::fill_f64((double*)ghh, 0.0, n * n, s));
    if ((rc = realq_hessian_accum(ctx, st->Xhat, st->s, T, n, (double*)ghh))) return rc;
    if ((rc = gram_accum(ctx, st->Xhat, st->X, st->s, T, n, (double*)gdh, (double*)gdd))) return rc;
    Timed tm(ctx, "init");
    RQ_HIP(ctx, realq::fill_f32(st->mA, 0.f, m * n, s));
    RQ_HIP(ctx, realq::fill_f32(st->vA, 0.f, m * n, s));
    RQ_HIP(ctx, realq::fill_u16(st->Dhi, 0, m * ldn, s));
    RQ_HIP(ctx, realq::fill_u16(st->Dlo, 0, m * ldn, s));
    RQ_HIP(ctx, realq::split_f64((const double*)ghh, st->Ghi, st->Glo, ldn, n, n, s));
    double* Ad = (double*)A;
    double* Ed = (double*)E;
    RQ_HIP(ctx, realq::widen_f32(st->W0, Ad, m * n, s));
    RQ_HIP(ctx, realq::dgemm(Ad, n, (const double*)gdh, n, Ed, n, m, n, n, false, s));
    RQ_HIP(ctx, realq::narrow_f64(Ed, st->C0, m * n, s));
    RQ_HIP(ctx, realq::dgemm(Ad, n, (const double*)gdd, n, Ed, n, m, n, n, false, s));
    RQ_HIP(ctx, realq::dot_f64(Ed, Ad, m * n, (double*)parts, s));
    RQ_HIP(ctx, realq::reduce_partials((const double*)parts, np, 1.0, st->cconst, s));
    st->t = 0;
    st->locked = 0;
    return REALQ_OK;
}

// P = D G_hh on columns [p0, n) (three MFMA passes: D_hi G_hi + D_lo G_hi + D_hi G_lo).
static int gram_product(realq_ctx* ctx, realq_bgd_state* st, int64_t p0) {
    const int64_t m = st->m, n = st->n, ldn = st->ldn, pw = n - p0;
    if (pw <= 0) return REALQ_OK;
    Timed tm(ctx, "gram_step");
    realq::GemmArgs g{st->Dhi, st->Dlo, ldn, st->Ghi + p0 * ldn, ldn, m, pw, n, 1};
    RQ_HIP(ctx, realq::gemm_store_f32(g, st->Pm + p0, n, 0, 1.f, ctx->stream));
    realq::GemmArgs g2{st->Dhi, nullptr, ldn, st->Glo + p0 * ldn, ldn, m, pw, n, 1};
    RQ_HIP(ctx, realq::gemm_acc_f32(g2, st->Pm + p0, n, 1.f, ctx->stream));
    return REALQ_OK;
}

// L = (c + sum (2 C0 + P) (W - W0)) / 2T with P over all columns.
static int gram_loss(realq_ctx* ctx, realq_bgd_state* st, const double* W, double* loss_out) {
    const int64_t np = realq::dot_f64_partials();
    void* parts;
    int rc;
    if ((rc = get_ws(ctx, "b_gparts", (size_t)(np + 1) * 8, &parts))) return rc;
    RQ_HIP(ctx, realq::dot_gram(st->C0, st->Pm, W, st->W0, st->m * st->n, (double*)parts, ctx->stream));
    RQ_HIP(ctx, hipMemcpyAsync((double*)parts + np, st->cconst, 8, hipMemcpyDeviceToDevice, ctx->stream));
    RQ_HIP(ctx, realq::reduce_partials((const double*)parts, np + 1, 0.5 / (double)st->T, loss_out, ctx->stream));
    return REALQ_OK;
}

static int check_state_args(realq_ctx* ctx, const float* W0, const uint16_t* X, const uint16_t* Xhat, int64_t m,
                            int64_t n, int64_t T, const realq_bgd_params* params, const float* M, const float* P) {
    if (m <= 0 || n <= 0 || T <= 0) return set_error(ctx, REALQ_ERR_SHAPE, "bgd state: need m, n, T > 0");
    if (!W0 || !X || !Xhat) return set_error(ctx, REALQ_ERR_INVALID_ARG, "bgd state: NULL W0, X or Xhat");
    int rc = validate_bgd(ctx, params);
    if (rc) return rc;
    const bool clip = params->loss_clip > 0.f, minib = params->batch > 0 && params->batch < T;
    if (params->form == REALQ_BGD_GRAM && (clip || minib))
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "the Gram form takes neither loss_clip nor a batch smaller than T");
    if (clip && (M || P))
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "loss_clip needs the identity metric (no M, no window partner P)");
    return REALQ_OK;
}

int realq_bgd_state_create(realq_ctx* ctx, realq_bgd_state** out, const float* W0, const uint16_t* X,
                           const uint16_t* Xhat, const float* s, const float* M, const float* P, int64_t m, int64_t n,
                           int64_t T, const realq_bgd_params* params) {
    if (!ctx || !out) return REALQ_ERR_INVALID_ARG;
    *out = nullptr;
    int rc = check_state_args(ctx, W0, X, Xhat, m, n, T, params, M, P);
    if (rc) return rc;
    realq_bgd_state* st = new (std::nothrow) realq_bgd_state();
    if (!st) return set_error(ctx, REALQ_ERR_OOM, "host allocation");
    st->ctx = ctx;
    st->m = m;
    st->n = n;
    st->T = T;
    st->W0 = W0;
    st->X = X;
    st->Xhat = Xhat;
    st->s = s;
    st->M = M;
    st->P = P;
    st->prm = *params;
    st->owns = true;
    rc = state_init(st);
    if (rc) {
        state_free(st);
        delete st;
        return rc;
    }
    *out = st;
    return REALQ_OK;
}

void realq_bgd_state_destroy(realq_bgd_state* st) {
    if (!st) return;
    state_free(st);
    delete st;
}

// ============================================================================ a3-a6: one column block

extern "C++" {
int realq::validate_q(realq_ctx* ctx, const realq_qparams* qp) {
    if (!qp) return set_error(ctx, REALQ_ERR_INVALID_ARG, "NULL qparams");
    if (qp->bits < 2 || qp->bits > 4) return set_error(ctx, REALQ_ERR_INVALID_ARG, "bits must be 2, 3 or 4");
    if (qp->group < 0) return set_error(ctx, REALQ_ERR_INVALID_ARG, "group must be >= 1, or 0 for one group per row");
    if (qp->block < 1 || qp->block > 128) return set_error(ctx, REALQ_ERR_INVALID_ARG, "block must be in 1..128");
    if (qp->grid < 1 || qp->grid > 100) return set_error(ctx, REALQ_ERR_INVALID_ARG, "grid must be in 1..100");
    if (qp->group > 0 && qp->block % qp->group != 0 && qp->group % qp->block != 0)
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "block and group must divide one another");
    if (qp->sym != 0 && qp->sym != 1) return set_error(ctx, REALQ_ERR_INVALID_ARG, "sym must be 0 or 1");
    if (!(qp->damp > 0.f) || !std::isfinite(qp->damp))
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "damp must be finite and > 0");
    return REALQ_OK;
}
}  // extern "C++"

// Rows [r0, r1) of one column block: search, quantize and compensate inside the block, then the
// trailing update; with a state, its copy of W - W0 follows on those rows.
static int quantize_rows(realq_ctx* ctx, double* W, int64_t m, int64_t n, int64_t r0, int64_t r1, int64_t c0,
                         int64_t bs, const float* U, const uint8_t* dead, const realq_qparams* qp, uint8_t* codes,
                         float* scales, uint8_t* zeros, realq_bgd_state* st) {
    int rc = validate_q(ctx, qp);
    if (rc) return rc;
    if (m <= 0 || n <= 0) return set_error(ctx, REALQ_ERR_SHAPE, "quantize_block: need m, n > 0");
    if (r0 < 0 || r1 <= r0 || r1 > m) return set_error(ctx, REALQ_ERR_SHAPE, "quantize_block: need 0 <= r0 < r1 <= m");
    if (c0 < 0 || bs < 1 || bs > 128 || c0 + bs > n)
        return set_error(ctx, REALQ_ERR_SHAPE, "quantize_block: need 0 <= c0, 1 <= bs <= 128, c0 + bs <= n");
    if (c0 % qp->block != 0 || (bs != qp->block && c0 + bs != n))
        return set_error(ctx, REALQ_ERR_SHAPE, "quantize_block: the block must be a whole column block of the sweep");
    if (!W || !U || !codes || !scales || !zeros)
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "quantize_block: NULL W, U, codes, scales or zeros");
    if (st && (st->m != m || st->n != n))
        return set_error(ctx, REALQ_ERR_SHAPE, "quantize_block: state shape differs from W");
    if (st && st->locked != c0)
        return set_error(ctx, REALQ_ERR_SHAPE, "quantize_block: blocks must be quantized in column order");
    if (st) {  // the trailing update changes D: the next step starts a block
        st->inc_c1 = -1;
        st->inc_ready = false;
    }
    const int64_t mr = r1 - r0;
    const int64_t group = qp->group > 0 ? qp->group : n;  // 0: one group per row
    const int64_t ngroups = (n + group - 1) / group;
    void* E;
    if ((rc = get_ws(ctx, "q_E", (size_t)mr * bs * 8, &E))) return rc;
    hipStream_t s = ctx->stream;
    realq::QuantArgs q{};
    q.W = W + r0 * n;
    q.m = mr;
    q.n = n;
    q.c0 = c0;
    q.bs = bs;
    q.U = U;
    q.dead = dead;
    q.bits = qp->bits;
    q.group = (int)group;
    q.grid = qp->grid;
    q.sym = qp->sym;
    q.codes = codes + r0 * n;
    q.scales = scales + r0 * ngroups;
    q.zeros = zeros + r0 * ngroups;
    q.ngroups = ngroups;
    q.E = (double*)E;
    q.W0 = st ? st->W0 + r0 * n : nullptr;
    q.Dhi = st ? st->Dhi + r0 * st->ldn : nullptr;
    q.Dlo = st ? st->Dlo + r0 * st->ldn : nullptr;
    q.ldd = st ? st->ldn : 0;
    {
        Timed tm(ctx, "quantize");
        RQ_HIP(ctx, realq::quantize_block(q, s));
    }
    const int64_t c1 = c0 + bs;
    if (c1 < n) {
        realq::ObsArgs a{};
        a.E = (const double*)E;
        a.lde = bs;
        a.U = U + c0 * n + c1;
        a.ldu = n;
        a.W = W + r0 * n + c1;
        a.ldw = n;
        a.M = mr;
        a.N = n - c1;
        a.K = bs;
        if (st) {
            a.W0 = st->W0 + r0 * n + c1;
            a.ldw0 = n;
            a.Dhi = st->Dhi + r0 * st->ldn + c1;
            a.Dlo = st->Dlo + r0 * st->ldn + c1;
            a.ldd = st->ldn;
        }
        Timed tm(ctx, "obs");
        RQ_HIP(ctx, realq::obs_update(a, s));
    }
    return REALQ_OK;
}

// The block's quantized weights stay locked (Sec. 4.3): B += (W_hat - W0)[:, block] Xhat[:, block]^T
// (the Gram form keeps no residual base and only moves the boundary).
static int lock_block(realq_ctx* ctx, realq_bgd_state* st, int64_t c0, int64_t bs) {
    const int64_t n = st->n;
    if (c0 != st->locked || bs < 1 || c0 + bs > n)
        return set_error(ctx, REALQ_ERR_SHAPE, "bgd_lock_block: blocks must be locked in column order");
    st->inc_c1 = -1;  // the residual base moves: the next step starts a block
    st->inc_ready = false;
    if (!st->gram) {
        realq::GemmArgs g{st->Dhi + c0, st->Dlo + c0, st->ldn, st->Xg + c0, st->ldx, st->m, st->at.count, bs, 1};
        Timed tm(ctx, "lock");
        RQ_HIP(ctx, realq::gemm_acc_f32(g, st->B, st->Tp, 1.f, ctx->stream));
    }
    st->locked = c0 + bs;
    return REALQ_OK;
}

int realq_quantize_block(realq_ctx* ctx, double* W, int64_t m, int64_t n, int64_t c0, int64_t bs, const float* U,
                         const uint8_t* dead, const realq_qparams* qp, uint8_t* codes, float* scales, uint8_t* zeros,
                         realq_bgd_state* st) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    int rc = quantize_rows(ctx, W, m, n, 0, m, c0, bs, U, dead, qp, codes, scales, zeros, st);
    if (rc) return rc;
    return st ? lock_block(ctx, st, c0, bs) : REALQ_OK;
}

int realq_quantize_block_rows(realq_ctx* ctx, double* W, int64_t m, int64_t n, int64_t r0, int64_t r1, int64_t c0,
                              int64_t bs, const float* U, const uint8_t* dead, const realq_qparams* qp,
                              uint8_t* codes, float* scales, uint8_t* zeros, realq_bgd_state* st) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    return quantize_rows(ctx, W, m, n, r0, r1, c0, bs, U, dead, qp, codes, scales, zeros, st);
}

int realq_bgd_lock_block(realq_ctx* ctx, realq_bgd_state* st, int64_t c0, int64_t bs) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    if (!st) return set_error(ctx, REALQ_ERR_INVALID_ARG, "bgd_lock_block: NULL state");
    return lock_block(ctx, st, c0, bs);
}

// ============================================================================ a7-a9: one BGD step

int realq_bgd_step(realq_ctx* ctx, realq_bgd_state* st, double* W, int64_t c1, float alpha, double* loss_out) {
    if (!ctx || !st) return REALQ_ERR_INVALID_ARG;
    if (!W) return set_error(ctx, REALQ_ERR_INVALID_ARG, "bgd_step: NULL W");
    if (c1 < 0 || c1 > st->n) return set_error(ctx, REALQ_ERR_SHAPE, "bgd_step: need 0 <= c1 <= n");
    if (!std::isfinite(alpha) || alpha < 0.f || alpha > 1.f)
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "bgd_step: alpha must lie in [0, 1]");
    const int64_t m = st->m, n = st->n, T = st->T, Tc = st->Tc, nJ = n - c1, ldn = st->ldn, ldx = st->ldx, Tp = st->Tp;
    hipStream_t s = ctx->stream;
    if (nJ == 0) {
        if (loss_out) RQ_HIP(ctx, realq::fill_f64(loss_out, NAN, 1, s));
        return REALQ_OK;
    }
    const bool dense = st->M || (st->P && alpha < 1.f);
    const bool clip = st->prm.loss_clip > 0.f;
    int rc;
    void *Gp = nullptr, *Gacc = nullptr;
    int64_t splits_used = 1;
    // tokens of this step: mini-batch (t mod nbatch) of the module's Adam step t (1-based), cut
    // into chunks; the plan sizes the split-K and loss-partial workspaces for every chunk
    const realq::plan::StepPlan pl = realq::plan::plan_step(m, nJ, T, st->Tb, Tc, st->t, ctx->cus,
                                                            clip ? realq::clip_apply_partials() : 0);
    // increments (token form): a later step of the block takes the change of its residual as
    // Q = bf16(Dacc) Xhat_J^T, its gradient as G0 + bf16(Q o s) Xhat_J and its loss as
    // L0 + <G0, bf16(Dacc)> / T + sum s Q^2 / 2T; the block's first step writes L0 and G0 and
    // restarts Dacc
    // (a caller taking more than `steps` steps at one c1 gets a fresh first step every `steps`
    // steps, so the displacement bound of the gate holds)
    const bool inc_step = st->inc && !st->gram && st->inc_c1 == c1 && st->inc_ready &&
                          st->inc_taken < (int64_t)st->prm.steps - 1;
    const bool inc_first = st->inc && !st->gram && !inc_step;
    const int64_t Tn = pl.Tn;
    const int64_t nchunks = (int64_t)pl.chunks.size();
    if (st->gram) {
        // gradient (1/T) M_a (C0 + D G_hh)[:, J]; the loss needs D G_hh on every column
        const bool want_loss = loss_out && !dense;
        if ((rc = get_ws(ctx, "b_G", (size_t)m * nJ * 4, &Gacc))) return rc;
        if ((rc = gram_product(ctx, st, want_loss ? 0 : c1))) return rc;
        if (loss_out) {
            if (dense) RQ_HIP(ctx, realq::fill_f64(loss_out, NAN, 1, s));
            else if ((rc = gram_loss(ctx, st, W, loss_out))) return rc;
        }
        RQ_HIP(ctx, realq::gram_grad(st->C0, st->Pm, n, c1, m, nJ, (float*)Gacc, s));
    } else {
        void* parts;
        if ((rc = get_ws(ctx, "b_Gp", (size_t)pl.gp_slices * m * nJ * 4, &Gp))) return rc;
        if (nchunks > 1 || dense)
            if ((rc = get_ws(ctx, "b_G", (size_t)m * nJ * 4, &Gacc))) return rc;
        if ((rc = get_ws(ctx, "b_parts", (size_t)pl.parts_total * 8, &parts))) return rc;
        double* const pbase = (double*)parts;
        const bool via_acc = nchunks > 1 || dense;
        // a later step's gradient GEMM gives the change since the block's first: that one is
        // added back (in Adam, or as the start of the accumulated gradient)
        if (inc_step && via_acc)
            RQ_HIP(ctx, hipMemcpyAsync(Gacc, st->G0, (size_t)m * nJ * 4, hipMemcpyDeviceToDevice, s));

        for (int64_t ch = 0; ch < nchunks; ++ch) {
            const int64_t t0 = pl.chunks[ch].t0, cur = pl.chunks[ch].len;
            double* const pch = pbase + pl.chunks[ch].parts_off;
            const int64_t pos = realq::plan::place_of(st->at, t0);
            const float* sc = st->sg ? st->sg + pos : nullptr;
            realq::GemmArgs g{st->Dhi + c1, st->Dlo + c1, ldn, st->Xg + pos * ldx + c1, ldx, m, cur, nJ, 1};
            if (inc_step) {
                realq::GemmArgs gi{st->Dinc + c1, nullptr, ldn, st->Xg + pos * ldx + c1, ldx, m, cur, nJ, 1};
                Timed tm(ctx, "resid_inc");
                RQ_HIP(ctx, realq::gemm_resid_inc(gi, sc, st->Rhi, q_ld(cur), pch, s));
            } else if (!clip) {
                Timed tm(ctx, "resid");
                RQ_HIP(ctx, realq::gemm_resid(g, st->B + pos, Tp, sc, st->Rhi, nullptr,
                                              r_ld(cur), pch, s, true));
            } else {
                // residual kept whole, per-token thresholds over the m channels, then the
                // clipped, weighted split for the gradient GEMM and the loss partials
                Timed tm(ctx, "resid");
                RQ_HIP(ctx, realq::gemm_resid_f32(g, st->B + pos, Tp, st->Rf, q_ld(cur), s));
                const int64_t k = std::max<int64_t>(1, (int64_t)std::ceil((double)st->prm.loss_clip * (double)m));
                RQ_HIP(ctx, realq::clip_select(st->Rf, q_ld(cur), m, cur, std::min(k, m), st->tau, s));
                RQ_HIP(ctx, realq::clip_apply(st->Rf, q_ld(cur), m, cur, st->tau, sc, st->Rhi,
                                              st->Rlo, pch, s));
            }
            {
                realq::GemmArgs g{st->Rhi, clip ? st->Rlo : st->Rhi + 32, clip ? q_ld(cur) : r_ld(cur),
                                  st->XhT + c1 * Tp + pos, Tp, m, nJ, cur, pl.splits};
                g.a_blocked = clip ? 0 : 1;
                if (inc_step) {  // bf16(Q o s) alone, row-major
                    g.Alo = nullptr;
                    g.lda = q_ld(cur);
                    g.a_blocked = 0;
                }
                splits_used = realq::gemm_effective_splits(cur, pl.splits);
                Timed tm(ctx, inc_step ? "grad_inc" : "grad");
                RQ_HIP(ctx, realq::gemm_grad(g, (float*)Gp, nJ, m * nJ, s));
            }
            if (via_acc) {
                // Gacc (+)= sum of this chunk's split slices, chunks in order
                RQ_HIP(ctx, realq::reduce_splits((const float*)Gp, splits_used, m, nJ, 1.f, (float*)Gacc,
                                                 ch > 0 || inc_step, s));
            }
        }
        if (inc_first && via_acc)
            RQ_HIP(ctx, hipMemcpyAsync(st->G0, Gacc, (size_t)m * nJ * 4, hipMemcpyDeviceToDevice, s));
        // the identity-metric loss of the block's first step (its partials exist for any metric: a
        // caller may change alpha between the steps of one block)
        if (inc_first) RQ_HIP(ctx, realq::reduce_partials(pbase, pl.parts_total, 0.5 / (double)Tn, st->L0, s));
        if (loss_out) {
            if (dense) {
                RQ_HIP(ctx, realq::fill_f64(loss_out, NAN, 1, s));
            } else if (inc_step) {
                void* dots;
                if ((rc = get_ws(ctx, "b_incdots", (size_t)realq::inc_loss_partials() * 8, &dots))) return rc;
                RQ_HIP(ctx, realq::inc_loss(st->L0, st->G0, st->Dinc + c1, ldn, m, nJ, pbase, pl.parts_total,
                                            (double)Tn, (double*)dots, loss_out, s));
            } else {
                RQ_HIP(ctx, realq::reduce_partials(pbase, pl.parts_total, 0.5 / (double)Tn, loss_out, s));
            }
        }
    }
    st->t += 1;
    realq::AdamArgs a{};
    a.W = W;
    a.W0 = st->W0;
    a.mA = st->mA;
    a.vA = st->vA;
    a.Dhi = st->Dhi;
    a.Dlo = st->Dlo;
    a.m = m;
    a.n = n;
    a.c1 = c1;
    a.ldd = ldn;
    a.Gp = (const float*)Gp;
    a.splits = splits_used;
    a.gscale = (float)(1.0 / (double)Tn);
    a.lr = st->prm.lr;
    a.beta1 = st->prm.beta1;
    a.beta2 = st->prm.beta2;
    a.eps = st->prm.eps;
    a.bc1 = (float)(1.0 / (1.0 - std::pow((double)st->prm.beta1, (double)st->t)));
    a.bc2 = (float)(1.0 / (1.0 - std::pow((double)st->prm.beta2, (double)st->t)));
    if (st->inc && !st->gram) {
        a.Dacc = st->Dacc;
        a.Dinc = st->Dinc;
        a.inc_reset = inc_first ? 1 : 0;
        a.G0 = st->G0;
        a.g0_mode = (nchunks > 1 || dense) ? 0 : (inc_first ? 1 : 2);
        st->inc_c1 = c1;
        st->inc_ready = true;
        st->inc_taken = inc_first ? 0 : st->inc_taken + 1;
    }
    if (!dense && nchunks == 1 && !st->gram) {
        Timed tm(ctx, "adam");
        RQ_HIP(ctx, realq::adam_update(a, s));
    } else if (!dense) {
        a.Gp = (const float*)Gacc;
        a.splits = 1;
        Timed tm(ctx, "adam");
        RQ_HIP(ctx, realq::adam_update(a, s));
    } else {
        // G = (1/T) M_a Gacc with M_a = alpha M + (1 - alpha) P (M = I when absent; Eq. slide_window),
        // on the matrix cores: M_a as a bf16 pair formed once per alpha (one per column block),
        // Gacc transposed and split; hi*hi + lo*hi in one launch, hi*lo accumulated in a second
        // (the lo*lo term is below float32 rounding of the product).
        if (!st->Mah) {
            void* p;
            if ((rc = state_alloc(st, &p, (size_t)m * realq::plan::row_stride(m) * 2, "s_Mah"))) return rc;
            st->Mah = (uint16_t*)p;
            if ((rc = state_alloc(st, &p, (size_t)m * realq::plan::row_stride(m) * 2, "s_Mal"))) return rc;
            st->Mal = (uint16_t*)p;
            st->Ma_alpha = -1.f;
        }
        if (st->Ma_alpha != alpha) {
            RQ_HIP(ctx, realq::blend_split(st->M, alpha < 1.f ? st->P : nullptr, alpha, m, st->Mah, st->Mal,
                                           realq::plan::row_stride(m), s));
            st->Ma_alpha = alpha;
        }
        void *Gm, *gth, *gtl;
        if ((rc = get_ws(ctx, "b_Gm", (size_t)m * nJ * 4, &Gm))) return rc;
        if ((rc = get_ws(ctx, "b_GTh", (size_t)realq::plan::row_stride(m) * nJ * 2, &gth))) return rc;
        if ((rc = get_ws(ctx, "b_GTl", (size_t)realq::plan::row_stride(m) * nJ * 2, &gtl))) return rc;
        const float invT = (float)(1.0 / (double)Tn);
        const int64_t mp = realq::plan::row_stride(m);
        {
            Timed tm(ctx, "metric");
            RQ_HIP(ctx,
                   realq::transpose_split_f32((const float*)Gacc, nJ, (uint16_t*)gth, (uint16_t*)gtl, mp, m, nJ, s));
            realq::GemmArgs g1{st->Mah, st->Mal, mp, (const uint16_t*)gth, mp, m, nJ, m, 1};
            RQ_HIP(ctx, realq::gemm_store_f32(g1, (float*)Gm, nJ, 0, invT, s));
            realq::GemmArgs g2{st->Mah, nullptr, mp, (const uint16_t*)gtl, mp, m, nJ, m, 1};
            RQ_HIP(ctx, realq::gemm_acc_f32(g2, (float*)Gm, nJ, invT, s));
        }
        Timed tm(ctx, "adam");
        RQ_HIP(ctx, realq::adam_update_dense(a, (const float*)Gm, s));
    }
    return REALQ_OK;
}

int realq_bgd_loss(realq_ctx* ctx, realq_bgd_state* st, const double* W, double* loss_out) {
    if (!ctx || !st) return REALQ_ERR_INVALID_ARG;
    if (!W || !loss_out) return set_error(ctx, REALQ_ERR_INVALID_ARG, "bgd_loss: NULL W or loss_out");
    if (st->M) return set_error(ctx, REALQ_ERR_SHAPE, "bgd_loss: only the identity metric is supported");
    if (st->gram) {
        int rc = gram_product(ctx, st, 0);
        if (rc) return rc;
        return gram_loss(ctx, st, W, loss_out);
    }
    // R = B + (W - W0)[:, J] Xhat[:, J]^T with J the columns not yet folded into B.
    // Places without a token hold zero inputs and a zero base: R is zero there.
    const int64_t m = st->m, T = st->T, n = st->n, c1 = st->locked, nJ = n - c1, ldn = st->ldn, ldx = st->ldx;
    int64_t nparts = 0;
    const std::vector<realq::plan::Chunk> chunks =
        realq::plan::plan_loss(m, st->at.count, st->at.apart ? st->at.chunk : st->Tc, &nparts);
    void* parts;
    int rc;
    if ((rc = get_ws(ctx, "b_parts", (size_t)nparts * 8, &parts))) return rc;
    if (nJ > 0) RQ_HIP(ctx, realq::split_diff_f64(W + c1, n, st->W0 + c1, n, st->Dhi + c1, st->Dlo + c1, ldn, m, nJ,
                                                  ctx->stream));
    for (const auto& c : chunks) {
        realq::GemmArgs g{st->Dhi + c1, st->Dlo + c1, ldn, st->Xg + c.t0 * ldx + c1, ldx, m, c.len, nJ, 1};
        RQ_HIP(ctx, realq::gemm_loss(g, st->B + c.t0, st->Tp, st->sg ? st->sg + c.t0 : nullptr,
                                     (double*)parts + c.parts_off, ctx->stream));
    }
    RQ_HIP(ctx, realq::reduce_partials((const double*)parts, nparts, 0.5 / (double)T, loss_out, ctx->stream));
    return REALQ_OK;
}

// ============================================================================ a10: window partner and hand-off

int realq_pullback_metric(realq_ctx* ctx, const float* W_next, const float* M_next, int64_t m_next, int64_t m,
                          int accumulate, float* P) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    if (m_next <= 0 || m <= 0) return set_error(ctx, REALQ_ERR_SHAPE, "pullback_metric: need m_next, m > 0");
    if (!W_next || !P) return set_error(ctx, REALQ_ERR_INVALID_ARG, "pullback_metric: NULL W_next or P");
    hipStream_t s = ctx->stream;
    // Float32 operands as three bf16 terms (all 24 bits), the product from the six term pairs above
    // its own float32 rounding.  A bf16 checkpoint's weights are exact in the first term: the
    // launches of the other pairs then find the flag down and return (the flag stays on the device,
    // the call asynchronous).  M = NULL: W^T W is symmetric, one triangle is formed.
    // 14336 x 4096 bf16-exact weights: 8.7 ms as a float32 vector GEMM (55 TFLOP/s), now 0.40 ms;
    // error against float64 1.7e-6 -> 2.7e-7 (shorter float32 sums).
    const int64_t kp = realq::plan::operand_stride(m_next);
    struct Terms {
        uint16_t *hi, *lo, *lo2;
    };
    int rc;
    if (realq::plan::pullback_small(m_next, m, M_next != nullptr)) {
        void* T = nullptr;
        if (M_next && (rc = get_ws(ctx, "p_T1", (size_t)m_next * m * 8, &T))) return rc;
        RQ_HIP(ctx, realq::pullback_f64(W_next, M_next, m_next, m, (double*)T, accumulate != 0, P, s));
        return REALQ_OK;
    }
    auto terms = [&](const char* slot, int64_t rows, Terms& t) -> int {
        void* p;
        if ((rc = get_ws(ctx, slot, (size_t)3 * rows * kp * 2, &p))) return rc;
        t.hi = (uint16_t*)p;
        t.lo = t.hi + rows * kp;
        t.lo2 = t.lo + rows * kp;
        return REALQ_OK;
    };
    void* flag;
    if ((rc = get_ws(ctx, "p_flag", 8, &flag))) return rc;
    RQ_HIP(ctx, realq::fill_f64((double*)flag, 0.0, 1, s));
    Terms w, r;
    if ((rc = terms("p_W", m, w))) return rc;
    RQ_HIP(ctx, realq::transpose_split3_f32(W_next, m, w.hi, w.lo, w.lo2, kp, m_next, m, (int*)flag, s));
    auto product = [&](const Terms& a, const Terms& b, int64_t N, const int* f, bool sym, bool acc, float* C,
                       int64_t ldc) -> int {
        realq::GemmArgs g[4] = {{a.hi, nullptr, kp, b.hi, kp, m, N, m_next, 1},
                                {a.hi, nullptr, kp, b.lo2, kp, m, N, m_next, 1},
                                {a.hi, a.lo, kp, b.lo, kp, m, N, m_next, 1},
                                {a.lo, a.lo2, kp, b.hi, kp, m, N, m_next, 1}};
        return sum_products(ctx, g, 4, f ? 1 : 4, f, sym, 0, acc, C, ldc);
    };
    if (!M_next) return product(w, w, m, (const int*)flag, true, accumulate != 0, P, m);
    // (M W)^T = W^T M^T [m, m_next], K-contiguous for the second product
    void* T1;
    if ((rc = terms("p_M", m_next, r))) return rc;
    RQ_HIP(ctx, realq::split3_f32(M_next, m_next, r.hi, r.lo, r.lo2, kp, m_next, m_next, nullptr, s));
    // float32 here; 8 bytes a value, so that a small call (in float64) after a larger one finds its room
    if ((rc = get_ws(ctx, "p_T1", (size_t)m * kp * 8, &T1))) return rc;
    if ((rc = product(w, r, m_next, nullptr, false, false, (float*)T1, kp))) return rc;
    if ((rc = terms("p_R", m, r))) return rc;
    RQ_HIP(ctx, realq::split3_f32((const float*)T1, kp, r.hi, r.lo, r.lo2, kp, m, m_next, nullptr, s));
    return product(w, r, m, nullptr, false, accumulate != 0, P, m);
}

int realq_handoff(realq_ctx* ctx, const float* Wa, const float* Wb, const uint16_t* X, int64_t T, int64_t n,
                  int64_t m, uint16_t* Y) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    if (T < 0 || n <= 0 || m <= 0) return set_error(ctx, REALQ_ERR_SHAPE, "handoff: need T >= 0, n, m > 0");
    if (T == 0) return REALQ_OK;
    if (!Wa || !X || !Y) return set_error(ctx, REALQ_ERR_INVALID_ARG, "handoff: NULL Wa, X or Y");
    hipStream_t s = ctx->stream;
    void *hi, *lo, *xg, *G = nullptr;
    int rc;
    const int64_t ldn = (n + 7) / 8 * 8;  // 16-byte operand rows whatever n is
    if ((rc = get_ws(ctx, "h_wh", (size_t)m * ldn * 2, &hi))) return rc;
    if ((rc = get_ws(ctx, "h_wl", (size_t)m * ldn * 2, &lo))) return rc;
    if (Wb && (rc = get_ws(ctx, "h_gate", (size_t)T * m * 4, &G))) return rc;
    const uint16_t* Xg = X;
    int64_t ldx = n;
    if (ldn != n) {  // without room for the copy the product takes the caller's rows, slower
        const size_t bytes = (size_t)T * ldn * 2;
        rc = ctx->ws["h_xg"].bytes < bytes && capturing(ctx) ? REALQ_ERR_OOM : get_ws(ctx, "h_xg", bytes, &xg);
        if (rc && rc != REALQ_ERR_OOM) return rc;
        if (!rc) {
            RQ_HIP(ctx, realq::copy_rows_u16(X, n, (uint16_t*)xg, ldn, T, n, s));
            Xg = (const uint16_t*)xg;
            ldx = ldn;
        }
    }
    // acc[i][t] = sum_j W[i][j] X[t][j], stored token-major
    realq::GemmArgs g{(const uint16_t*)hi, (const uint16_t*)lo, ldn, Xg, ldx, m, T, n, 1};
    if (!Wb) {
        RQ_HIP(ctx, realq::split_diff_f32(Wa, n, nullptr, 0, (uint16_t*)hi, (uint16_t*)lo, ldn, m, n, s));
        RQ_HIP(ctx, realq::gemm_store_bf16_t(g, Y, m, s));
        return REALQ_OK;
    }
    RQ_HIP(ctx, realq::split_diff_f32(Wa, n, nullptr, 0, (uint16_t*)hi, (uint16_t*)lo, ldn, m, n, s));
    RQ_HIP(ctx, realq::gemm_store_f32_t(g, (float*)G, m, s));  // gate pre-activation, token-major
    RQ_HIP(ctx, realq::split_diff_f32(Wb, n, nullptr, 0, (uint16_t*)hi, (uint16_t*)lo, ldn, m, n, s));
    RQ_HIP(ctx, realq::gemm_swiglu_t(g, (const float*)G, m, Y, m, s));
    return REALQ_OK;
}

// ============================================================================ a11 with a dense metric
// L = (1/2T) sum_t s_t R_t^T M R_t with R = W0 Delta^T + D Xhat^T (Delta = Xhat - X, D = W - W0)
// expands through the calibration Gram matrices G_dd = Delta^T S Delta, G_dh = Delta^T S Xhat
// and G_hh = Xhat^T S Xhat (the Hessian accumulator) into
//   2T L = <W0 G_dd, M W0> + 2 <W0 G_dh, M D> + <D G_hh, M D>,
// n x n token contractions plus m x n x n and m x m x n float64 products instead of an
// m x m x T contraction.  Every term is built from the small quantities Delta and D.
static int dense_final_loss(realq_ctx* ctx, const realq_layer_desc* d, const double* W, const double* Ghh,
                            double* loss_dev) {
    const int64_t m = d->m, n = d->n, T = d->T;
    hipStream_t s = ctx->stream;
    int rc;
    void *gdh, *gdd, *A, *D, *E, *MX, *M64, *parts;
    if ((rc = get_ws(ctx, "g_dh", (size_t)n * n * 8, &gdh))) return rc;
    if ((rc = get_ws(ctx, "g_dd", (size_t)n * n * 8, &gdd))) return rc;
    if ((rc = gram_accum(ctx, d->Xhat, d->X, d->s, T, n, (double*)gdh, (double*)gdd))) return rc;
    Timed tm(ctx, "dense_loss");
    const int64_t np = realq::dot_f64_partials();
    if ((rc = get_ws(ctx, "g_A", (size_t)m * n * 8, &A))) return rc;
    if ((rc = get_ws(ctx, "g_D", (size_t)m * n * 8, &D))) return rc;
    if ((rc = get_ws(ctx, "g_E", (size_t)m * n * 8, &E))) return rc;
    if ((rc = get_ws(ctx, "g_MX", (size_t)m * n * 8, &MX))) return rc;
    if ((rc = get_ws(ctx, "g_M", (size_t)m * m * 8, &M64))) return rc;
    if ((rc = get_ws(ctx, "g_parts", (size_t)4 * np * 8, &parts))) return rc;
    double* Ad = (double*)A;
    double* Dd = (double*)D;
    double* Ed = (double*)E;
    double* MXd = (double*)MX;
    double* pp = (double*)parts;
    RQ_HIP(ctx, realq::widen_f32(d->W0, Ad, m * n, s));
    RQ_HIP(ctx, realq::sub_f64_f32(W, d->W0, Dd, m * n, s));
    RQ_HIP(ctx, realq::widen_f32(d->M, (double*)M64, m * m, s));
    // <W0 G_dd, M W0>
    RQ_HIP(ctx, realq::dgemm(Ad, n, (const double*)gdd, n, Ed, n, m, n, n, false, s));
    RQ_HIP(ctx, realq::dgemm((const double*)M64, m, Ad, n, MXd, n, m, n, m, false, s));
    RQ_HIP(ctx, realq::dot_f64(Ed, MXd, m * n, pp, s));
    // 2 <W0 G_dh, M D>
    RQ_HIP(ctx, realq::dgemm(Ad, n, (const double*)gdh, n, Ed, n, m, n, n, false, s));
    RQ_HIP(ctx, realq::dgemm((const double*)M64, m, Dd, n, MXd, n, m, n, m, false, s));
    RQ_HIP(ctx, realq::dot_f64(Ed, MXd, m * n, pp + np, s));
    RQ_HIP(ctx, realq::dot_f64(Ed, MXd, m * n, pp + 2 * np, s));
    // <D G_hh, M D>
    RQ_HIP(ctx, realq::dgemm(Dd, n, Ghh, n, Ed, n, m, n, n, false, s));
    RQ_HIP(ctx, realq::dot_f64(Ed, MXd, m * n, pp + 3 * np, s));
    RQ_HIP(ctx, realq::reduce_partials(pp, 4 * np, 0.5 / (double)T, loss_dev, s));
    return REALQ_OK;
}

// ============================================================================ a1-a11: whole module

int realq_quantize_layer(realq_ctx* ctx, const realq_layer_desc* d, realq_layer_out* out) {
    if (!ctx) return REALQ_ERR_INVALID_ARG;
    if (!d || !out) return set_error(ctx, REALQ_ERR_INVALID_ARG, "quantize_layer: NULL desc or out");
    int rc = validate_q(ctx, &d->q);
    if (rc) return rc;
    if ((rc = check_state_args(ctx, d->W0, d->X, d->Xhat, d->m, d->n, d->T, &d->bgd, d->M, d->P))) return rc;
    if (!out->codes || !out->scales || !out->zeros || !out->W_hat)
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "quantize_layer: NULL codes, scales, zeros or W_hat");
    const int64_t m = d->m, n = d->n, T = d->T;
    const bool grouped = d->s_groups != nullptr;
    if (!grouped && d->n_groups != 0)
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "quantize_layer: n_groups needs s_groups (0 without)");
    if (grouped && (d->n_groups < 1 || d->n_groups > m))
        return set_error(ctx, REALQ_ERR_INVALID_ARG, "quantize_layer: need 1 <= n_groups <= m");
    // row groups of rsz rows (one group of all m rows without s_groups); ngr of them hold rows
    const int64_t rsz = grouped ? (m + d->n_groups - 1) / d->n_groups : m;
    const int64_t ngr = (m + rsz - 1) / rsz;
    hipStream_t s = ctx->stream;
    realq::EventPair ev;
    RQ_HIP(ctx, ev.create());
    RQ_HIP(ctx, hipEventRecord(ev.a, s));

    // a1-a2: Hessian and inverse factor of every row group (each factorisation synchronises once)
    void *Hacc, *Uw = out->U, *deadw = out->dead;
    if ((rc = get_ws(ctx, "l_H", (size_t)n * n * 8, &Hacc))) return rc;
    if (!Uw && (rc = get_ws(ctx, "l_U", (size_t)ngr * n * n * 4, &Uw))) return rc;
    if (!deadw && (rc = get_ws(ctx, "l_dead", (size_t)ngr * n, &deadw))) return rc;
    for (int64_t g = 0; g < ngr; ++g) {
        RQ_HIP(ctx, realq::fill_f64((double*)Hacc, 0.0, n * n, s));
        const float* sg = grouped ? d->s_groups + g * T : d->s;
        if ((rc = realq_hessian_accum(ctx, d->Xhat, sg, T, n, (double*)Hacc))) return rc;
        if ((rc = realq_chol_inverse(ctx, (const double*)Hacc, n, T, d->q.damp, out->H ? out->H + g * n * n : nullptr,
                                     (float*)Uw + g * n * n, (uint8_t*)deadw + g * n)))
            return rc;
    }

    // state on context workspaces (reused across calls of the same size)
    realq_bgd_state st;
    st.ctx = ctx;
    st.m = m;
    st.n = n;
    st.T = T;
    st.W0 = d->W0;
    st.X = d->X;
    st.Xhat = d->Xhat;
    st.s = d->s;
    st.M = d->M;
    st.P = d->P;
    st.prm = d->bgd;
    st.owns = false;
    const bool bgd = d->bgd.steps > 0;
    if (bgd && (rc = state_init(&st))) return rc;

    // float64 working weights; W_hat receives their float32 rounding at the end
    void* Ww;
    if ((rc = get_ws(ctx, "l_W", (size_t)m * n * 8, &Ww))) return rc;
    double* W = (double*)Ww;
    RQ_HIP(ctx, realq::widen_f32(d->W0, W, m * n, s));
    const int64_t nb = (n + d->q.block - 1) / d->q.block;
    if (out->loss_trace && bgd) RQ_HIP(ctx, realq::fill_f64(out->loss_trace, NAN, nb * d->bgd.steps, s));
    for (int64_t b = 0; b < nb; ++b) {
        const int64_t c0 = b * d->q.block, bs = std::min<int64_t>(d->q.block, n - c0), c1 = c0 + bs;
        char rname[48];
        snprintf(rname, sizeof(rname), "block %lld (columns %lld..%lld)", (long long)b, (long long)c0,
                 (long long)(c1 - 1));
        realq::Range block_range(rname);
        for (int64_t g = 0; g < ngr; ++g) {
            if ((rc = quantize_rows(ctx, W, m, n, g * rsz, std::min(m, (g + 1) * rsz), c0, bs,
                                    (const float*)Uw + g * n * n, (const uint8_t*)deadw + g * n, &d->q, out->codes,
                                    out->scales, out->zeros, bgd ? &st : nullptr)))
                return rc;
        }
        if (bgd && (rc = lock_block(ctx, &st, c0, bs))) return rc;
        if (!bgd || c1 >= n) continue;
        float alpha = 1.f;
        if (d->window_total > 1) {
            const double bg = (double)(d->window_offset + b + 1);
            alpha = (float)(1.0 - (bg - 1.0) / (double)(d->window_total - 1));
            alpha = std::min(1.f, std::max(0.f, alpha));
        }
        for (int k = 0; k < d->bgd.steps; ++k) {
            double* lo = out->loss_trace ? out->loss_trace + b * d->bgd.steps + k : nullptr;
            if ((rc = realq_bgd_step(ctx, &st, W, c1, alpha, lo))) return rc;
        }
    }
    // a11: final loss (own metric) at the quantized weights
    out->loss_final = NAN;
    void* lf;
    if ((rc = get_ws(ctx, "l_loss", 8, &lf))) return rc;
    if (!d->M) {
        if (!bgd) {
            // no state yet: build the residual base once for the loss
            st.prm.tok_chunk = d->bgd.tok_chunk;
            if ((rc = state_init(&st))) return rc;
        }
        if ((rc = realq_bgd_loss(ctx, &st, W, (double*)lf))) return rc;
    } else {
        if (grouped) {  // the loss weighs tokens by s, not by a row group's saliency
            RQ_HIP(ctx, realq::fill_f64((double*)Hacc, 0.0, n * n, s));
            if ((rc = realq_hessian_accum(ctx, d->Xhat, d->s, T, n, (double*)Hacc))) return rc;
        }
        if ((rc = dense_final_loss(ctx, d, W, (const double*)Hacc, (double*)lf))) return rc;
    }
    RQ_HIP(ctx, realq::narrow_f64(W, out->W_hat, m * n, s));
    RQ_HIP(ctx, hipEventRecord(ev.b, s));
    RQ_HIP(ctx, hipMemcpyAsync(&out->loss_final, lf, 8, hipMemcpyDeviceToHost, s));
    RQ_HIP(ctx, hipStreamSynchronize(s));
    float ms = 0.f;
    RQ_HIP(ctx, hipEventElapsedTime(&ms, ev.a, ev.b));
    out->ms_total = ms;
    if ((rc = realq::harvest(ctx))) return rc;
    if (!std::isfinite(out->loss_final))
        return set_error(ctx, REALQ_ERR_NONFINITE,
                         "quantize_layer: the final loss is not finite (NaN or Inf in W0, X, s or the metric)");
    return REALQ_OK;
}

}  // extern "C"
