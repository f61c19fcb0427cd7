// Quantization of one column block (Alg. 1 inner loop; Sec. 3.2 Eq. gptq_update).
//
// One wave64 owns one weight row; lane l holds block columns l and l+64 in registers.  Per row:
//   1. dead columns of the block are zeroed;
//   2. when a quantization group starts (a group may span the whole row), its
//      (scale, zero) pair is searched in float64 over the shrink factors p_k = 1 - k/100
//      and all zero points: the least error wins, errors up to
//      least * (1 + 2^-40) + 2^-60 * sum x^2 form one tie, and among a tie the least
//      (k, |z - z_nat|, z), with z_nat = rint(-lo maxq / (hi - lo)); the symmetric
//      quantizer takes the range [-max|x|, max|x|] and only the zero point (maxq + 1) / 2
//      (search_group says which candidates need scoring);
//   3. columns are quantized in order with the scale as stored (float32):
//      q = clamp(rint(w/s) + z, 0, maxq) decided in float64, w_hat = s (q - z) (exact in
//      float64, so the float32 output is the float32 dequantization of the stored
//      parameters), and the error
//      e = (w - w_hat) / U_jj is propagated to the block's later columns with row j of
//      the inverse factor U (held in LDS);
//
//   4. w_hat, codes, the block error E and the bf16 split of w_hat - W0 are written.
// Every float64 step that decides an integer (rint of x / s, the candidate errors, the natural
// zero) keeps the exact ties of the underlying arithmetic as ties: x / s comes from the correctly
// rounded reciprocal and one Newton correction, which leaves exact half-integers exact.
// The working weights are float64 (one row in registers, two values per lane): every
// later column takes up to 127 compensation updates here and more from the trailing
// update, Block-GD and later blocks, and a float32 running value would drift by
// about 1e-8, enough to move a few codes per module across a rounding boundary.
//
// obs_update_kernel then applies the trailing update W[:, c1:] -= E_b U[b, c1:]
// (Sec. 3.2) in float64 and refreshes the bf16 split of W - W0 for those columns.
#include "common.h"
#include "f64mma.h"
#include "kernels.h"

namespace realq {

namespace {
constexpr int QB = 128;          // maximum block width
constexpr int WAVES = 4;         // rows per workgroup, one wave each
constexpr int CACHE = 6;         // evaluated batches (64 candidates each) kept for the tie decision
constexpr int ALL_LEN = 4;       // groups of up to this many values have every candidate scored

constexpr double TIE_RTOL = 0x1p-40;  // search errors within TIE_RTOL * least + TIE_ATOL * sum x^2
constexpr double TIE_ATOL = 0x1p-60;  // are one tie

struct Best {
    int k, dist, z;
};

__device__ __forceinline__ bool better(const Best& a, const Best& b) {
    if (a.k != b.k) return a.k < b.k;
    if (a.dist != b.dist) return a.dist < b.dist;
    return a.z < b.z;
}

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
    return v;
}

// a / b from y = 1/b (correctly rounded): one Newton correction of a*y.  An exact quotient, a
// half-integer among them, comes out exact; an infinite a*y is the quotient's own overflow.
__device__ __forceinline__ double div_by(double a, double b, double y) {
    const double q = a * y;
    const double c = fma(fma(-q, b, a), y, q);
    return fabs(q) < INFINITY ? c : q;
}

// The wave's own LDS: the values being searched, the candidates waiting for a full batch, and the
// errors of the evaluated batches.
struct WaveMem {
    double x[QB];
    double err[CACHE * 64];
    uint16_t id[CACHE * 64];
    uint16_t wait[128];
};

// LDS traffic between lanes of one wave completes in order; this keeps the compiler from moving it.
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Values of one group: in the wave's LDS (len <= QB), or streamed through it from a row of W.
struct GroupSrc {
    const double* row;   // first value in memory, or NULL when the values already sit in LDS
    const uint8_t* dead; // flags of the streamed columns (may be NULL)
    int64_t len;
};

// Calls f(x) for every value in order, x uniform over the wave.
template <class F>
__device__ __forceinline__ void for_values(const GroupSrc& g, WaveMem& wm, int lane, F f) {
    if (!g.row) {
        const int n = (int)g.len;
        int e = 0;
        for (; e + 4 <= n; e += 4) {
            const double x0 = wm.x[e], x1 = wm.x[e + 1], x2 = wm.x[e + 2], x3 = wm.x[e + 3];
            f(x0);
            f(x1);
            f(x2);
            f(x3);
        }
        for (; e < n; ++e) f(wm.x[e]);
        return;
    }
    for (int64_t e0 = 0; e0 < g.len; e0 += QB) {
        wave_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t e = e0 + 64 * h + lane;
            if (e < g.len) wm.x[64 * h + lane] = (g.dead && g.dead[e]) ? 0.0 : g.row[e];
        }
        wave_sync();
        const int cnt = (int)min((int64_t)QB, g.len - e0);
        for (int e = 0; e < cnt; ++e) f(wm.x[e]);
    }
}

struct Range2 {  // the two least and two greatest values, and the sum of squares
    double lo, lo2, hi, hi2, ss;
};

__device__ __forceinline__ Range2 value_range(const GroupSrc& g, const WaveMem& wm, int lane) {
    double lo = INFINITY, lo2 = INFINITY, hi = -INFINITY, hi2 = -INFINITY, ss = 0.0;
    for (int64_t e = lane; e < g.len; e += 64) {
        const double x = g.row ? ((g.dead && g.dead[e]) ? 0.0 : g.row[e]) : wm.x[e];
        lo2 = fmin(lo2, fmax(lo, x));
        lo = fmin(lo, x);
        hi2 = fmax(hi2, fmin(hi, x));
        hi = fmax(hi, x);
        ss = fma(x, x, ss);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double l = __shfl_xor(lo, off), l2 = __shfl_xor(lo2, off);
        const double h = __shfl_xor(hi, off), h2 = __shfl_xor(hi2, off);
        lo2 = fmin(fmin(lo2, l2), fmax(lo, l));
        lo = fmin(lo, l);
        hi2 = fmax(fmax(hi2, h2), fmin(hi, h));
        hi = fmax(hi, h);
        ss += __shfl_xor(ss, off);
    }
    return {lo, lo2, hi, hi2, ss};
}

}  // namespace

// Every candidate of a group scored in one walk over its values: lane l takes zero points
// (l % 4) * (MAXQ + 1) / 4 and on, and of every 16 shrink factors number l / 4; the quotient of a value
// and a scale serves all the lane's zeros.  About 130 operations a value for 1280 candidates, where 64
// candidates a batch take 11.  best: the winner by the tie rule.
template <int MAXQ, int R>
__device__ __forceinline__ Best search_all(const GroupSrc& g, WaveMem& wm, int grid, double span, double ss, int znat,
                                           int lane) {
#pragma clang fp contract(off)
    constexpr int ZL = (MAXQ + 1) / 4;
    const int z0 = (lane & 3) * ZL;
    double s[R], y[R], e[R][ZL], lo[ZL], hi[ZL];
#pragma unroll
    for (int u = 0; u < ZL; ++u) {
        lo[u] = (double)(-(z0 + u));
        hi[u] = (double)(MAXQ - (z0 + u));
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int k = 16 * r + (lane >> 2);
        s[r] = k < grid ? ((1.0 - (double)k / 100.0) * span) / (double)MAXQ : 1.0;
        y[r] = 1.0 / s[r];
#pragma unroll
        for (int u = 0; u < ZL; ++u) e[r][u] = 0.0;
    }
    for_values(g, wm, lane, [&](double x) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double q = rint(div_by(x, s[r], y[r]));
#pragma unroll
            for (int u = 0; u < ZL; ++u) {
                const double d = x - s[r] * fmin(fmax(q, lo[u]), hi[u]);
                e[r][u] = fma(d, d, e[r][u]);
            }
        }
    });
    double emin = INFINITY;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < ZL; ++u)
            if (16 * r + (lane >> 2) < grid) emin = fmin(emin, e[r][u]);
    const double thr = wave_min(emin) * (1.0 + TIE_RTOL) + TIE_ATOL * ss;
    Best best{1 << 30, 1 << 30, 1 << 30};
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < ZL; ++u) {
            const Best c{16 * r + (lane >> 2), abs(z0 + u - znat), z0 + u};
            if (c.k < grid && e[r][u] <= thr && better(c, best)) best = c;
        }
    return best;
}

// Joint (scale, zero) search of one group by one wave; the result is in all lanes.
//
// Every candidate's error is the float64 sum over the group's values in order, so the decision is
// that of scoring all grid x (MAXQ + 1) candidates; but most of them cannot win, and are not scored.
// The clipping error of the group's two least and two greatest values alone bounds a candidate's
// error from below.  A first batch of 64 candidates around the natural zero gives an error the
// winner cannot exceed; the candidates whose bound is above it are dropped (bounds carry a 1e-9
// margin for their own rounding), and the rest are packed into batches of 64, one per lane.  Of
// 1280 candidates about 100 to 200 are scored on Gaussian groups.  The tie rule needs every error up to the
// final threshold: the first CACHE batches are kept in LDS, and a search that needed more goes
// through the surviving candidates once more.
// ALL: where more than CACHE batches would be scored, and for groups of up to ALL_LEN values, all
// candidates are, in one walk (search_all): the four extreme values say little about the sum of a long
// group, and a few values are scored sooner than bounds are formed.
template <int MAXQ, bool ALL>
__device__ __forceinline__ void search_group(const GroupSrc& g, WaveMem& wm, int grid, bool sym, int lane,
                                             double& scale, int& zero) {
#pragma clang fp contract(off)
    constexpr int ZSYM = (MAXQ + 1) / 2;
    const Range2 r = value_range(g, wm, lane);
    double lo = fmin(0.0, r.lo), hi = fmax(0.0, r.hi);
    if (sym) {
        const double amax = fmax(-lo, hi);
        lo = -amax;
        hi = amax;
    }
    if (lo == hi) {
        lo = -1.0;
        hi = 1.0;
    }
    const double span = hi - lo;
    // the shrink factor cancels from -p_k lo / s_k: one natural zero for every k
    const double fnat = (-lo * (double)MAXQ) / span;
    const int znat = (int)fmin(fmax(rint(fnat), 0.0), (double)MAXQ);
    int zalt = fnat > (double)znat ? znat + 1 : znat - 1;  // the next nearest zero
    if (zalt < 0) zalt = 1;
    if (zalt > MAXQ) zalt = MAXQ - 1;

    // error of candidate (k, z) over the group, one candidate per lane
    auto score = [&](int k, int z) {
        const double p = 1.0 - (double)k / 100.0;
        const double s = (p * span) / (double)MAXQ;
        const double y = 1.0 / s;
        // s * clamp(q, -z, maxq - z) is clamp(s q, -s z, s (maxq - z)): rounding is monotone
        const double bl = s * (double)(-z), bh = s * (double)(MAXQ - z);
        double e = 0.0;
        for_values(g, wm, lane, [&](double x) {
            const double v = s * rint(div_by(x, s, y));
            const double d = x - fmin(fmax(v, bl), bh);
            e = fma(d, d, e);
        });
        return e;
    };
    const int zbits = sym ? 0 : (MAXQ == 15 ? 4 : (MAXQ == 7 ? 3 : 2));
    const int total = grid << zbits;
    auto k_of = [&](int id) { return id >> zbits; };
    auto z_of = [&](int id) { return sym ? ZSYM : id & MAXQ; };
    // candidates of the first batch: the least 64 shrink factors, or 32 of them with the two zeros
    // nearest the natural one
    auto seeded = [&](int k, int z) { return sym ? k < 64 : (k < 32 && (z == znat || z == zalt)); };
    const double below = (1.0 - 1e-9);
    auto bound = [&](int k, int z) {
        const double s = (1.0 - 0.01 * (double)k) * span * (1.0 / (double)MAXQ);
        const double bl = -s * (double)z, bh = s * (double)(MAXQ - z);
        const double a = fmax(bl - r.lo, 0.0), b = fmax(r.hi - bh, 0.0);
        const double c = fmax(bl - r.lo2, 0.0), d = fmax(r.hi2 - bh, 0.0);
        double e = fma(a, a, b * b);
        if (g.len > 1) e = fma(c, c, fma(d, d, e));
        return e * below;
    };
    auto threshold = [&](double emin) { return emin * (1.0 + TIE_RTOL) + TIE_ATOL * r.ss; };

    double emin = INFINITY;
    int batches = 0;
    // score one candidate per lane (id < 0: none; the lane still takes part in streaming the values)
    // and keep it
    auto batch = [&](int id) {
        const int c = id < 0 ? 0 : id;
        const double e = score(k_of(c), z_of(c));
        emin = fmin(emin, wave_min(id < 0 ? INFINITY : e));
        if (batches < CACHE) {
            wm.err[batches * 64 + lane] = id >= 0 ? e : NAN;  // no candidate passes no threshold
            wm.id[batches * 64 + lane] = (uint16_t)c;
        }
        ++batches;
    };
    auto survives = [&](int id, bool skip_seeded, double thr) {
        const int k = k_of(id), z = z_of(id);
        return id < total && !(skip_seeded && seeded(k, z)) && !(bound(k, z) > thr);
    };
    // walk the remaining candidates in order and hand full batches of the surviving ones to f
    auto survivors = [&](bool skip_seeded, auto thr, auto f) {
        int n = 0;
        for (int id0 = 0; id0 < total; id0 += 64) {
            const int id = id0 + lane;
            const bool keep = survives(id, skip_seeded, thr());
            const uint64_t mask = __ballot(keep);
            if (keep) wm.wait[n + __popcll(mask & ((1ull << lane) - 1))] = (uint16_t)id;
            n += __popcll(mask);
            wave_sync();
            if (n >= 64) {
                const int take = wm.wait[lane];
                const uint16_t rest = wm.wait[64 + lane];
                wave_sync();
                wm.wait[lane] = rest;
                wave_sync();
                n -= 64;
                f(take);
            }
        }
        if (n > 0) f(lane < n ? (int)wm.wait[lane] : -1);
    };
    Best best{1 << 30, 1 << 30, 1 << 30};
    bool all = ALL && g.len <= ALL_LEN;
    if (!all) {
        const int k = sym ? lane : (lane & 31);
        const int z = lane < 32 ? znat : zalt;
        batch(k < grid ? (sym ? k : (k << zbits) + z) : -1);
    }
    if (ALL && !all) {  // the walk below drops these and, as emin falls, more
        int n = 0;
        for (int id0 = 0; id0 < total; id0 += 64) n += __popcll(__ballot(survives(id0 + lane, true, threshold(emin))));
        all = n > (CACHE - 1) * 64;
    }
    if (ALL && all) {
        best = grid <= 80 ? search_all<MAXQ, 5>(g, wm, grid, span, r.ss, znat, lane)
                          : search_all<MAXQ, 7>(g, wm, grid, span, r.ss, znat, lane);
    } else {
        survivors(true, [&] { return threshold(emin); }, batch);
        const double thr = threshold(emin);
        auto offer = [&](double e, int id) {
            const Best c{k_of(id), abs(z_of(id) - znat), z_of(id)};
            if (e <= thr && better(c, best)) best = c;
        };
        wave_sync();
        if (ALL || batches <= CACHE) {
            for (int b = 0; b < batches; ++b) offer(wm.err[b * 64 + lane], wm.id[b * 64 + lane]);
        } else {
            survivors(false, [&] { return thr; }, [&](int id) {
                const int c = id < 0 ? 0 : id;
                const double e = score(k_of(c), z_of(c));
                if (id >= 0) offer(e, c);
            });
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        Best o;
        o.k = __shfl_xor(best.k, off);
        o.dist = __shfl_xor(best.dist, off);
        o.z = __shfl_xor(best.z, off);
        if (better(o, best)) best = o;
    }
    const double p = 1.0 - (double)best.k / 100.0;
    scale = (p * span) / (double)MAXQ;
    zero = best.z;
}

// One wave per row, so that a module of m rows has m waves whatever its size (four rows one after
// the other on a wave left three quarters of the chip idle below 4096 rows and the search took
// 20 scored candidates and two divisions per value and lane: 486 us a block at 512 rows, 491 us at
// 4096; now 63 and 141 us).  The row's column loop is a serial chain of about 17 dependent float64
// operations per column (the quantizer's quotient and the compensation's through precomputed
// reciprocals, no division in the chain); the block's triangle of U sits in LDS, packed by rows.
template <int MAXQ, bool ALL>
__global__ __launch_bounds__(WAVES * 64) void quantize_block_kernel(QuantArgs q) {
    __shared__ float sU[QB * (QB + 1) / 2];
    __shared__ double sR[QB];  // 1 / U_jj
    __shared__ WaveMem mem[WAVES];
    const int bs = (int)q.bs;
    const int64_t c0 = q.c0, n = q.n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // row a of the triangle starts at a * bs - a (a - 1) / 2 and holds columns a .. bs - 1
    for (int a = wave; a < bs; a += WAVES) {
        const float* u = q.U + (c0 + a) * n + c0;
        float* d = sU + a * bs - a * (a - 1) / 2 - a;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int b = 64 * h + lane;
            if (b >= a && b < bs) d[b] = u[b];
        }
    }
    __syncthreads();
    for (int a = threadIdx.x; a < bs; a += WAVES * 64) sR[a] = 1.0 / (double)sU[a * bs - a * (a - 1) / 2];
    __syncthreads();

    const int64_t i = (int64_t)blockIdx.x * WAVES + wave;
    if (i >= q.m) return;  // no block-level barrier below
    WaveMem& wm = mem[wave];
    const int64_t group = q.group;
    double* Wrow = q.W + i * n;
    const bool in0 = lane < bs, in1 = lane + 64 < bs;
    double w0 = in0 ? Wrow[c0 + lane] : 0.0;
    double w1 = in1 ? Wrow[c0 + 64 + lane] : 0.0;
    if (q.dead) {
        if (in0 && q.dead[c0 + lane]) w0 = 0.0;
        if (in1 && q.dead[c0 + 64 + lane]) w1 = 0.0;
    }
    double scale = 1.0, zf = 0.0;
    if (c0 % group != 0) {  // group started in an earlier block: reuse its parameters
        const int64_t g = c0 / group;
        scale = (double)q.scales[i * q.ngroups + g];
        zf = (double)q.zeros[i * q.ngroups + g];
    }
    double inv = 1.0 / scale;
    double e0 = 0.0, e1 = 0.0;
    uint8_t code0 = 0, code1 = 0;
    for (int j0 = 0; j0 < bs;) {
        // columns j0 .. jn - 1 share one group
        const int64_t in_group = (c0 + j0) % group;
        const int jn = (int)min((int64_t)bs, j0 + group - in_group);
        if (in_group == 0) {
            // ---- (scale, zero) search over the group's current values
            GroupSrc src{nullptr, nullptr, min(group, n - (c0 + j0))};
            if (j0 + src.len <= bs) {  // whole group inside the block: from the registers
                wave_sync();
                if (lane >= j0 && lane < j0 + src.len) wm.x[lane - j0] = w0;
                if (lane + 64 >= j0 && lane + 64 < j0 + src.len) wm.x[lane + 64 - j0] = w1;
                wave_sync();
            } else {  // it extends past the block (only at j0 == 0): the untouched row
                src.row = Wrow + c0;
                src.dead = q.dead ? q.dead + c0 : nullptr;
            }
            int zi;
            search_group<MAXQ, ALL>(src, wm, q.grid, q.sym != 0, lane, scale, zi);
            scale = (double)(float)scale;  // the stored float32 scale is the one used
            zf = (double)zi;
            inv = 1.0 / scale;
            if (lane == 0) {
                q.scales[i * q.ngroups + (c0 + j0) / group] = (float)scale;
                q.zeros[i * q.ngroups + (c0 + j0) / group] = (uint8_t)zi;
            }
        }
        // ---- quantize the columns in order, each compensated on the block's later ones
        auto column = [&](int j, double wj, auto own) {
            const float* u = sU + j * bs - j * (j - 1) / 2 - j;
            const double ujj = (double)u[j], rj = sR[j];
            const double u0 = in0 && lane > j ? (double)u[lane] : 0.0;
            const double u1 = in1 && lane + 64 > j ? (double)u[lane + 64] : 0.0;
            const double qv = fmin(fmax(rint(div_by(wj, scale, inv)) + zf, 0.0), (double)MAXQ);
            const double wq = scale * (qv - zf);
            const double err = div_by(wj - wq, ujj, rj);
            own(wq, err, (uint8_t)qv);
            if (lane > j && in0) w0 = fma(-err, u0, w0);
            if (lane + 64 > j && in1) w1 = fma(-err, u1, w1);
        };
        for (int j = j0; j < min(jn, 64); ++j)
            column(j, bcast(w0, j), [&](double wq, double err, uint8_t c) {
                if (lane == j) {
                    w0 = wq;
                    e0 = err;
                    code0 = c;
                }
            });
        for (int j = max(j0, 64); j < jn; ++j)
            column(j, bcast(w1, j - 64), [&](double wq, double err, uint8_t c) {
                if (lane == j - 64) {
                    w1 = wq;
                    e1 = err;
                    code1 = c;
                }
            });
        j0 = jn;
    }
    // ---- write back
    if (in0) {
        const int64_t c = c0 + lane;
        Wrow[c] = w0;
        q.codes[i * n + c] = code0;
        q.E[i * bs + lane] = e0;
        if (q.Dhi) {
            uint16_t h, l;
            split_bf16((float)(w0 - (double)q.W0[i * n + c]), h, l);
            q.Dhi[i * q.ldd + c] = h;
            q.Dlo[i * q.ldd + c] = l;
        }
    }
    if (in1) {
        const int64_t c = c0 + 64 + lane;
        Wrow[c] = w1;
        q.codes[i * n + c] = code1;
        q.E[i * bs + 64 + lane] = e1;
        if (q.Dhi) {
            uint16_t h, l;
            split_bf16((float)(w1 - (double)q.W0[i * n + c]), h, l);
            q.Dhi[i * q.ldd + c] = h;
            q.Dlo[i * q.ldd + c] = l;
        }
    }
}

hipError_t quantize_block(const QuantArgs& q, hipStream_t st) {
    if (q.m <= 0 || q.bs <= 0) return hipSuccess;
    const unsigned grid = (unsigned)((q.m + WAVES - 1) / WAVES);
    // In groups of more than two blocks most candidates may survive their bounds, and those of a few
    // columns are too short for bounds to pay: both may score every candidate in one walk.  Groups
    // in between keep the kernel without it (161 registers instead of 227; 256 columns a group 5.6 ms and
    // 5.9 with it, 16 a group 7.6 and 8.9); the symmetric search has one zero point and at most 100
    // candidates.  Quantizer of plain GPTQ, 4096 x 4096, asymmetric: one group a row 27.5 ms without it,
    // 8.1 with; 1024 columns a group 15.3 and 8.0; 512 8.3 and 7.2; one column a group 68.8 and 40.5.
    const bool all = !q.sym && (q.group > 2 * QB || q.group <= ALL_LEN);
    switch (q.bits) {
#define RQ_CASE(b)                                                                                 \
    case b:                                                                                        \
        if (all)                                                                                   \
            hipLaunchKernelGGL((quantize_block_kernel<(1 << b) - 1, true>), dim3(grid), dim3(WAVES * 64), 0, st, q);  \
        else                                                                                       \
            hipLaunchKernelGGL((quantize_block_kernel<(1 << b) - 1, false>), dim3(grid), dim3(WAVES * 64), 0, st, q); \
        break;
        RQ_CASE(2)
        RQ_CASE(3)
        RQ_CASE(4)
#undef RQ_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- trailing update, float64
// W -= E U on the float64 matrix cores, one 64 x 64 tile of W per workgroup (small enough that a
// 512-row module still has a workgroup per 64 rows, and at 4096 x 2048 the 2048 tiles fill the
// chip).  K is at most the block width, so a tile reads 96 KB of E and U from cache for 64 KB of W
// moved: bound by the read and write of W once the chip is full (4096 rows, 2048 columns on average:
// 103 -> 64 us against 4 x 4 vector tiles; 512 x 256: 40 -> 22 us).
__global__ __launch_bounds__(256) void obs_update_kernel(ObsArgs a, int64_t tiles_n, int vec_e, int vec_u) {
    using F = F64Tile<64>;
    __shared__ __attribute__((aligned(16))) double lds[4 * F::LDS];
    const int64_t m0 = (blockIdx.x / tiles_n) * 64, n0 = (blockIdx.x % tiles_n) * 64;
    f64x4 acc[F::SUB][F::SUB];
    F::product<true, false>(acc, lds, 0, a.K,
                            F64CheckKC<double>{a.E + m0 * a.lde, a.lde, a.M - m0, a.K, vec_e != 0},
                            F64CheckOC<float>{a.U + n0, a.ldu, a.N - n0, a.K, vec_u != 0});
    F::each(acc, [&](int r, int c, double x) {
        const int64_t i = m0 + r, j = n0 + c;
        if (i >= a.M || j >= a.N) return;
        double* w = a.W + i * a.ldw + j;
        const double v = *w - x;
        *w = v;
        if (a.Dhi) {
            uint16_t h, l;
            split_bf16((float)(v - (double)a.W0[i * a.ldw0 + j]), h, l);
            a.Dhi[i * a.ldd + j] = h;
            a.Dlo[i * a.ldd + j] = l;
        }
    });
}

hipError_t obs_update(const ObsArgs& a, hipStream_t st) {
    if (a.M <= 0 || a.N <= 0 || a.K <= 0) return hipSuccess;
    const int64_t tiles_m = (a.M + 63) / 64, tiles_n = (a.N + 63) / 64;
    const int vec_e = ((uintptr_t)a.E & 15) == 0 && a.lde % 2 == 0, vec_u = ((uintptr_t)a.U & 15) == 0 && a.ldu % 4 == 0;
    hipLaunchKernelGGL(obs_update_kernel, dim3((unsigned)(tiles_m * tiles_n)), dim3(256), 0, st, a, tiles_n, vec_e,
                       vec_u);
    return hipGetLastError();
}

}  // namespace realq
