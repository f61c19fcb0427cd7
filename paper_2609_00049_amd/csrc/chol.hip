// Inverse factor of the damped Hessian in float64 (Sec. 3.2; Alg. 1 "its inverse").
//
// GPTQ's compensation for column j uses row j of the inverse of H restricted to the
// columns not yet quantized.  Those rows, scaled, are the rows of the upper factor U
// with H_d^{-1} = U^T U.  With J the index reversal, A = J H_d J = L L^T (lower
// Cholesky) gives H_d^{-1} = (J L^{-1} J)^T (J L^{-1} J), so U = J L^{-1} J.
//
// Steps (all float64, products on the float64 matrix cores, f64mma.h):
//   prep     H = scale * H_acc; dead columns (H_jj == 0) get H_jj = 1; lambda = damp * mean(diag);
//            A = J (H + lambda I) J, padded to a multiple of 64 with identity.
//   Cholesky in outer panels of 256 columns.  Inside one, each 64-column panel is one launch
//            (chol_panel_kernel: update from the outer panel's earlier columns, factor and invert
//            the diagonal block, solve); after it, one symmetric update of the trailing matrix with
//            K = 256, so that matrix is read and written n / 256 times instead of n / 64.
//   inverse  X = L^{-1} by recursive doubling: with the aligned diagonal blocks of size s already
//            inverted (s = 64: the diagonal factor's own inverses), each aligned block of size 2s
//            [[L_A, 0], [L_CA, L_C]] gets its lower-left block X_CA = -X_C (L_CA X_A), two batched
//            float64 tile products per level that skip the tiles where a triangular operand is
//            zero; the intermediate L_CA X_A is parked, transposed, in the unused upper triangle of
//            the factor's work array.
//   U        U[i][j] = X[n-1-i][n-1-j] (j >= i), stored as float32.
//
// The diagonal blocks of L itself are not kept: the solve and the doubling need their inverses
// only.  Above X's diagonal blocks only the upper halves of its aligned 128-blocks are read, and
// the panels zero those: the work arrays need no clearing.
//
// Measured on an MI355X, this file's call alone: n = 512 1.35 -> 0.40 ms, n = 1024 2.68 -> 0.78 ms,
// n = 4096 12.6 -> 3.8 ms, n = 14336 141 -> 51 ms against 64-column panels with a launch each for the factor (118 us: column
// substitution by single threads over LDS), the solve and the update, and vector-FMA tiles.
#include "common.h"
#include "f64mma.h"
#include "kernels.h"

namespace realq {

namespace {
constexpr int NB = 64;        // panel width
constexpr int OUTER = 4;      // panels per outer panel
constexpr int SR = NB + 2;    // row stride of a row-major 64 x 64 block in LDS: rows 4 banks apart

typedef double (*Blk)[SR];
typedef double f64x2 __attribute__((ext_vector_type(2)));

// 16 x 16 product over k in [0, K): c + sign * A(16 rows from ra, columns from ka) * B, with
// B(k, j) = Bm[rb + j][kb + k] (BT) or Bm[kb + k][rb + j].
template <bool BT>
__device__ __forceinline__ f64x4 mma16(f64x4 c, Blk Am, int ra, int ka, Blk Bm, int rb, int kb, int K, double sign) {
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    for (int k = 0; k < K; k += 4) {
        const double a = sign * Am[ra + r][ka + k + g];
        const double b = BT ? Bm[rb + r][kb + k + g] : Bm[kb + k + g][rb + r];
        c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    return c;
}
__device__ __forceinline__ f64x4 get16(Blk M, int r0, int c0) {
    const int lane = threadIdx.x & 63;
    f64x4 c;
#pragma unroll
    for (int v = 0; v < 4; ++v) c[v] = M[r0 + 4 * v + (lane >> 4)][c0 + (lane & 15)];
    return c;
}
__device__ __forceinline__ void put16(Blk M, int r0, int c0, f64x4 c) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < 4; ++v) M[r0 + 4 * v + (lane >> 4)][c0 + (lane & 15)] = c[v];
}

// 1 / sqrt(d) for d > 0 to about an ulp: the hardware estimate and two Newton steps.
__device__ __forceinline__ double rsqrt64(double d) {
    double y = __builtin_amdgcn_rsq(d);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(y, fma(-0.5 * d * y, y, 0.5), y);
    return y;
}
}  // namespace

// ---------------------------------------------------------------- prep
// scratch[0] = lambda.  One block: deterministic mean of the fixed diagonal.
__global__ __launch_bounds__(1024) void chol_diag_kernel(const double* __restrict__ Hacc, int64_t n, double scale,
                                                         double damp, uint8_t* dead, double* scratch) {
    __shared__ double red[1024];
    double acc = 0.0;
    for (int64_t j = threadIdx.x; j < n; j += 1024) {
        double d = scale * Hacc[j * n + j];
        bool dd = d == 0.0;
        if (dead) dead[j] = dd ? 1 : 0;
        acc += dd ? 1.0 : d;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) scratch[0] = damp * (red[0] / (double)n);
}

// A = the index-reversed damped Hessian (padded with the identity), blocks on and below the
// diagonal only; nonfinite[0] = 1 when an entry of the accumulator is NaN or infinite (a non-finite
// input reached the Hessian).  One row per blockIdx.x, 1024 columns per block.
__global__ __launch_bounds__(256) void chol_fill_kernel(const double* __restrict__ Hacc, int64_t n, int64_t np,
                                                        double scale, const double* __restrict__ scratch,
                                                        double* __restrict__ A, float* Hout, int* nonfinite) {
    const double lam = scratch[0];
    const int64_t r = blockIdx.x, hr = n - 1 - r;
    bool bad = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t c = blockIdx.y * 1024 + u * 256 + threadIdx.x;
        if (c >= np) break;
        double v = r == c ? 1.0 : 0.0;
        if (r < n && c < n) {
            const int64_t hc = n - 1 - c;
            const double h = scale * Hacc[hr * n + hc];
            bad |= !isfinite(h);
            if (Hout) Hout[hr * n + hc] = (float)h;
            v = r == c ? (h == 0.0 ? 1.0 : h) + lam : h;
        }
        if (c / NB <= r / NB) A[r * np + c] = v;
    }
    if (bad) *nonfinite = 1;
}

// ---------------------------------------------------------------- one 64-column panel
// Workgroup b handles row block kb + b of column block kb; `first` is the outer panel's first
// block.  Every workgroup forms and factors the diagonal block for itself (the factor takes about
// 8 us of one compute unit and would otherwise be a launch of its own that all others wait for),
// workgroup 0 stores its inverse, the others their solved block L = P L_kk^{-T}.
//
// Bound by latency: per outer panel four dependent launches of 24 us and more (34 on average), 8 us of each
// the factor's 64 pivots (a reciprocal square root and the next column's update each, in the registers of one
// wave, 16 columns at a time with the rest of the block updated by all waves' matrix products).
__global__ __launch_bounds__(256) void chol_panel_kernel(double* __restrict__ A, int64_t np, int64_t kb, int64_t first,
                                                         double* __restrict__ X, int* flag) {
    __shared__ __attribute__((aligned(16))) double sL[NB][SR];
    __shared__ __attribute__((aligned(16))) double sV[NB][SR];
    __shared__ __attribute__((aligned(16))) double sP[NB][SR];
    __shared__ double sR[NB];  // reciprocal pivots
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t ti = kb + blockIdx.x;
    const bool own = ti != kb;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;  // this wave's 32 x 32 quarter
    const int lr = threadIdx.x >> 2, lc = (threadIdx.x & 3) * 16;  // 16 values of a row per thread

    f64x2 rl[8], rp[8];
    auto fetch = [&](int64_t cb) {
        const f64x2* l = reinterpret_cast<const f64x2*>(A + (kb * NB + lr) * np + cb * NB + lc);
        const f64x2* p = reinterpret_cast<const f64x2*>(A + (ti * NB + lr) * np + cb * NB + lc);
#pragma unroll
        for (int e = 0; e < 8; ++e) rl[e] = l[e];
#pragma unroll
        for (int e = 0; e < 8; ++e) rp[e] = p[e];  // the diagonal block once more in workgroup 0
    };
    auto stage = [&](Blk L, Blk P) {
#pragma unroll
        for (int e = 0; e < 8; ++e) *reinterpret_cast<f64x2*>(&L[lr][lc + 2 * e]) = rl[e];
#pragma unroll
        for (int e = 0; e < 8; ++e) *reinterpret_cast<f64x2*>(&P[lr][lc + 2 * e]) = rp[e];
    };
    // D = A_kk - sum L_k,p L_k,p^T and P = A_i,k - sum L_i,p L_k,p^T over the outer panel's blocks p
    f64x4 ad[2][2], ap[2][2];
    fetch(kb);
    stage(sL, sP);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            ad[i][j] = get16(sL, wr + 16 * i, wc + 16 * j);
            ap[i][j] = get16(sP, wr + 16 * i, wc + 16 * j);
        }
    if (first < kb) fetch(first);
    for (int64_t p = first; p < kb; ++p) {
        __syncthreads();
        stage(sV, sP);
        __syncthreads();
        if (p + 1 < kb) fetch(p + 1);
        const int r = lane & 15, g = lane >> 4;
#pragma unroll 4
        for (int k = 0; k < NB; k += 4) {
            double a[2], b[2], c[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = -sV[wr + 16 * i + r][k + g];
                b[i] = sV[wc + 16 * i + r][k + g];
                c[i] = -sP[wr + 16 * i + r][k + g];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    ad[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], ad[i][j], 0, 0, 0);
                    ap[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[i], b[j], ap[i][j], 0, 0, 0);
                }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            put16(sL, wr + 16 * i, wc + 16 * j, ad[i][j]);
            put16(sP, wr + 16 * i, wc + 16 * j, ap[i][j]);
        }
    __syncthreads();

    // factor D in 16-column steps: wave 0 eliminates the step's columns with one row per lane, then
    // all waves update the remaining lower blocks
    for (int b = 0; b < 4; ++b) {
        const int c0 = 16 * b;
        if (wave == 0) {
            double a[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) a[j] = sL[lane][c0 + j];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                double d = bcast(a[k], c0 + k);
                if (!(d > 0.0)) {  // not positive definite (or NaN): flag it and keep values finite
                    if (lane == 0) *flag = 1;
                    d = 1.0;
                }
                const double y = rsqrt64(d);
                if (lane == 0) sR[c0 + k] = y;
                a[k] = lane == c0 + k ? d * y : a[k] * y;
#pragma unroll
                for (int j = k + 1; j < 16; ++j) a[j] = fma(-a[k], bcast(a[k], c0 + j), a[j]);
            }
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (lane >= c0 + j) sL[lane][c0 + j] = a[j];
        }
        __syncthreads();
        // lower 16-blocks (i, j), b < j <= i, dealt to the waves
        int t = 0;
        for (int j = b + 1; j < 4; ++j)
            for (int i = j; i < 4; ++i, ++t)
                if ((t & 3) == wave)
                    put16(sL, 16 * i, 16 * j,
                          mma16<true>(get16(sL, 16 * i, 16 * j), sL, 16 * i, c0, sL, 16 * j, c0, 16, -1.0));
        __syncthreads();
    }
    // V = L^{-1}: the four 16-blocks on the diagonal, one column per lane, then by doubling
    for (int e = threadIdx.x; e < NB * NB; e += 256) sV[e >> 6][e & 63] = 0.0;
    __syncthreads();
    if (wave == 0) {
        const int b0 = (lane >> 4) * 16, c = lane & 15;
        double x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            double s = i == c ? 1.0 : 0.0;
#pragma unroll
            for (int k = 0; k < i; ++k) s = fma(-sL[b0 + i][b0 + k], x[k], s);
            x[i] = s * sR[b0 + i];
            sV[b0 + i][b0 + c] = x[i];  // exactly 0 above the diagonal
        }
    }
    __syncthreads();
    const f64x4 z4 = {0.0, 0.0, 0.0, 0.0};
    f64x4 t4 = z4;
    {  // 32-blocks: X10 = -X11 (L10 X00)
        const int o = 32 * (wave & 1);
        if (wave < 2) put16(sV, o, o + 16, mma16<false>(z4, sL, o + 16, o, sV, o, o, 16, 1.0));  // parked above
        __syncthreads();
        if (wave < 2) {
            put16(sV, o + 16, o, mma16<false>(z4, sV, o + 16, o + 16, sV, o + 16, o, 16, -1.0));
            put16(sV, o, o + 16, z4);
        }
        __syncthreads();
    }
    {  // the 64-block: one 16-block of the 32 x 32 products per wave
        const int i0 = 16 * (wave >> 1), j0 = 16 * (wave & 1);
        put16(sV, i0, 32 + j0, mma16<false>(z4, sL, 32 + i0, 0, sV, j0, 0, 32, 1.0));
        __syncthreads();
        t4 = mma16<false>(z4, sV, 32 + i0, 32, sV, 32 + j0, 0, 32, -1.0);
        put16(sV, 32 + i0, j0, t4);
        __syncthreads();
        put16(sV, i0, 32 + j0, z4);
        __syncthreads();
    }
    if (!own) {
        double* d = X + (kb * NB + lr) * np + kb * NB + lc;
#pragma unroll
        for (int e = 0; e < 8; ++e) reinterpret_cast<f64x2*>(d)[e] = *reinterpret_cast<f64x2*>(&sV[lr][lc + 2 * e]);
        if (kb % 2 == 0 && kb * NB + NB < np) {  // the 128-wide tiles of the inverse read this block
#pragma unroll
            for (int e = 0; e < 8; ++e) reinterpret_cast<f64x2*>(d + NB)[e] = f64x2{0.0, 0.0};
        }
        return;
    }
    // L_ik = P V^T
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) ap[i][j] = mma16<true>(z4, sP, wr + 16 * i, 0, sV, wc + 16 * j, 0, NB, 1.0);
    double* P = A + ti * NB * np + kb * NB;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                P[(wr + 16 * i + 4 * v + (lane >> 4)) * np + wc + 16 * j + (lane & 15)] = ap[i][j][v];
}

// ---------------------------------------------------------------- trailing update
// A22 -= L21 L21^T over K = 64 OUTER columns from k0, lower tiles of T x T.
template <int T>
__global__ __launch_bounds__(256, 2) void chol_syrk_kernel(double* __restrict__ A, int64_t np, int64_t k0, int64_t base) {
    using F = F64Tile<T>;
    __shared__ __attribute__((aligned(16))) double lds[4 * F::LDS];
    const int64_t t = blockIdx.x;
    int64_t ti = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
    while (ti * (ti + 1) / 2 > t) --ti;
    const int64_t tj = t - ti * (ti + 1) / 2;
    const int64_t ri = base + ti * T, rj = base + tj * T;
    f64x4 acc[F::SUB][F::SUB];
    const int li = (int)min((int64_t)T, np - ri), lj = (int)min((int64_t)T, np - rj);
    F::template product<true, true>(acc, lds, k0, base, F64LoadKC{A + ri * np, np, li}, F64LoadKC{A + rj * np, np, lj});
    double* C = A + ri * np + rj;
    F::each(acc, [&](int r, int c, double x) {
        if (r < li && c < lj) C[(int64_t)r * np + c] -= x;
    });
}

// ---------------------------------------------------------------- triangular inverse, one doubling level
// Pair p of the level joins the inverted blocks A = [off, off + s) and C = [off + s, off + s + Mp),
// off = 2 s p.  FIRST: the parked product, transposed, T1^T[j][i] = sum_k X_A[k][j] L_CA[i][k]
// (X_A lower triangular: k >= j), at the upper block's place in the factor's array.  Otherwise
// X_CA[i][j] = -sum_k X_C[i][k] T1[k][j] (k <= i).
template <int T, bool FIRST>
__global__ __launch_bounds__(256, 2) void chol_pair_kernel(double* __restrict__ A, double* __restrict__ X, int64_t np,
                                                        int64_t s) {
    using F = F64Tile<T>;
    __shared__ __attribute__((aligned(16))) double lds[4 * F::LDS];
    const int64_t off = blockIdx.z * 2 * s;
    const int64_t Mp = min(s, np - off - s);
    // rows walk the triangle's long side first: the largest K ranges start first
    const int64_t tr = FIRST ? blockIdx.y : gridDim.y - 1 - blockIdx.y;
    const int64_t r0 = tr * T, c0 = (int64_t)blockIdx.x * T;
    const int64_t rows = FIRST ? s : Mp, cols = FIRST ? Mp : s;
    if (r0 >= rows || c0 >= cols) return;
    double* const Xa = X + off * (np + 1);
    double* const Lca = A + (off + s) * np + off;
    double* const T1 = A + off * np + off + s;  // [j][i]
    double* const Xc = X + (off + s) * (np + 1);
    const int lr = (int)min((int64_t)T, rows - r0), lc = (int)min((int64_t)T, cols - c0);
    f64x4 acc[F::SUB][F::SUB];
    if constexpr (FIRST) {
        F::template product<false, true>(acc, lds, r0, s, F64LoadOC{Xa + r0, np, lr}, F64LoadKC{Lca + c0 * np, np, lc});
        F::each(acc, [&](int r, int c, double x) {
            if (r < lr && c < lc) T1[(r0 + r) * np + c0 + c] = x;
        });
    } else {
        F::template product<true, true>(acc, lds, 0, min(r0 + T, Mp), F64LoadKC{Xc + r0 * np, np, lr},
                                        F64LoadKC{T1 + c0 * np, np, lc});
        double* const out = X + (off + s + r0) * np + off + c0;
        F::each(acc, [&](int r, int c, double x) {
            if (r < lr && c < lc) out[(int64_t)r * np + c] = -x;
        });
    }
}

// One row of U per blockIdx.x, 1024 columns per block.
__global__ __launch_bounds__(256) void chol_extract_u_kernel(const double* __restrict__ X, int64_t np, int64_t n,
                                                             float* __restrict__ U) {
    const int64_t i = blockIdx.x;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t j = blockIdx.y * 1024 + u * 256 + threadIdx.x;
        if (j < n) U[i * n + j] = (j >= i) ? (float)X[(n - 1 - i) * np + (n - 1 - j)] : 0.f;
    }
}

hipError_t chol_inverse(const CholArgs& c, hipStream_t st) {
    const int64_t n = c.n, np = c.np;
    const int64_t nb = np / NB;
    auto wide = [](int64_t count) { return (unsigned)((count + 1023) / 1024); };
    hipLaunchKernelGGL(chol_diag_kernel, dim3(1), dim3(1024), 0, st, c.Hacc, n, c.scale, c.damp, c.dead, c.scratch);
    hipLaunchKernelGGL(chol_fill_kernel, dim3((unsigned)np, wide(np)), dim3(256), 0, st, c.Hacc, n, np, c.scale,
                       c.scratch, c.A, c.Hout, c.flag + 1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int64_t kb = 0; kb < nb; ++kb) {
        const int64_t first = kb / OUTER * OUTER;
        hipLaunchKernelGGL(chol_panel_kernel, dim3((unsigned)(nb - kb)), dim3(256), 0, st, c.A, np, kb, first, c.Linv,
                           c.flag);
        if (kb + 1 == first + OUTER && kb + 1 < nb) {
            // 128-wide tiles once they fill the chip; below that 64-wide ones (four times as many)
            const int64_t base = (kb + 1) * NB, rem = np - base, t128 = (rem + 127) / 128, t64 = rem / 64;
            if (t128 * (t128 + 1) / 2 >= 256)
                hipLaunchKernelGGL(chol_syrk_kernel<128>, dim3((unsigned)(t128 * (t128 + 1) / 2)), dim3(256), 0, st, c.A,
                                   np, first * NB, base);
            else
                hipLaunchKernelGGL(chol_syrk_kernel<64>, dim3((unsigned)(t64 * (t64 + 1) / 2)), dim3(256), 0, st, c.A,
                                   np, first * NB, base);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // X = L^{-1}: the diagonal 64-blocks came out of the factorisation; level s completes every
    // aligned 2s block (the last one cut at np) from its two inverted halves
    for (int64_t sz = NB; sz < np; sz *= 2) {
        const unsigned pairs = (unsigned)((np - sz + 2 * sz - 1) / (2 * sz));
        if (sz >= 128 && pairs * (sz / 128) * (sz / 128) >= 256) {  // as for the trailing update
            const unsigned t = (unsigned)(sz / 128);
            hipLaunchKernelGGL((chol_pair_kernel<128, true>), dim3(t, t, pairs), dim3(256), 0, st, c.A, c.Linv, np, sz);
            hipLaunchKernelGGL((chol_pair_kernel<128, false>), dim3(t, t, pairs), dim3(256), 0, st, c.A, c.Linv, np, sz);
        } else {
            const unsigned t = (unsigned)(sz / 64);
            hipLaunchKernelGGL((chol_pair_kernel<64, true>), dim3(t, t, pairs), dim3(256), 0, st, c.A, c.Linv, np, sz);
            hipLaunchKernelGGL((chol_pair_kernel<64, false>), dim3(t, t, pairs), dim3(256), 0, st, c.A, c.Linv, np, sz);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(chol_extract_u_kernel, dim3((unsigned)n, wide(n)), dim3(256), 0, st, c.Linv, np, n, c.U);
    return hipGetLastError();
}

}  // namespace realq
