// Memory-bound helper kernels: fills, bf16 transposes and splits, deterministic
// reductions and the fused split-K reduction + Adam update (Appendix D.1 constants
// arrive as arguments).  Every kernel here is HBM-bound; loops are grid-strided
// with coalesced rows.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace realq {

namespace {
constexpr int TB = 256;
inline unsigned grid_for(int64_t count, int per_thread = 1) {
    int64_t b = (count + (int64_t)TB * per_thread - 1) / ((int64_t)TB * per_thread);
    if (b < 1) b = 1;
    if (b > 65536) b = 65536;
    return (unsigned)b;
}
}  // namespace

template <class T>
__global__ void fill_kernel(T* p, T v, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t fill_f32(float* p, float v, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_kernel<float>, dim3(grid_for(count, 4)), dim3(TB), 0, st, p, v, count);
    return hipGetLastError();
}
hipError_t fill_f64(double* p, double v, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_kernel<double>, dim3(grid_for(count, 4)), dim3(TB), 0, st, p, v, count);
    return hipGetLastError();
}
hipError_t fill_u16(uint16_t* p, uint16_t v, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_kernel<uint16_t>, dim3(grid_for(count, 4)), dim3(TB), 0, st, p, v, count);
    return hipGetLastError();
}

// ---------------------------------------------------------------- tiled transposes (64 x 64 tiles via LDS)
// out[c][r] of a token-major bf16 array.  Bound by HBM: 16-byte loads along a row and 16-byte stores
// along a column where the arrays allow them (2-byte accesses per lane moved 2.4 TB/s), the 16-bit
// tile in LDS with rows 33 banks apart so that the eight values of a column chunk and the eight chunks
// of a wave fall on different banks.  1024 columns x 131072 tokens with the weighted terms: 622 us
// as two passes of 2-byte accesses, 245 us here.
// SCALE: also the three bf16 terms of s[r] * x (hi + lo + lo2 holds all 24 bits of the float32
// product), in the same pass over the input; o0 (the plain transpose) may then be NULL.
namespace {
struct TransposeArgs {
    const uint16_t* in;
    int64_t ldi;
    const float* s;
    uint16_t *o0, *hi, *lo, *lo2;
    int64_t ldo, rows, cols, tiles_c;
    int vec_in, vec_out;  // rows of the input / of every output 16-byte aligned
};
}  // namespace
template <bool SCALE>
__global__ __launch_bounds__(256) void transpose_kernel(TransposeArgs a) {
    __shared__ uint16_t tile[64][66];
    __shared__ float ts[64];
    const int64_t tr = blockIdx.x / a.tiles_c, tc = blockIdx.x % a.tiles_c;
    const int64_t r0 = tr * 64, c0 = tc * 64;
    const int t = threadIdx.x;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int rr = (t >> 3) + 32 * p, cc = (t & 7) * 8;
        const int64_t r = r0 + rr, c = c0 + cc;
        u16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (r < a.rows) {
            const uint16_t* q = a.in + r * a.ldi + c;
            if (a.vec_in && c + 8 <= a.cols) v = *reinterpret_cast<const u16x8*>(q);
            else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (c + e < a.cols) v[e] = q[e];
            }
        }
#pragma unroll
        for (int e = 0; e < 8; e += 2)
            *reinterpret_cast<uint32_t*>(&tile[rr][cc + e]) = (uint32_t)v[e] | ((uint32_t)v[e + 1] << 16);
    }
    if (SCALE && t < 64) ts[t] = r0 + t < a.rows ? a.s[r0 + t] : 0.f;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int cc = (t >> 3) + 32 * p, rr = (t & 7) * 8;
        const int64_t c = c0 + cc, r = r0 + rr;
        if (c >= a.cols || r >= a.rows) continue;
        const int64_t o = c * a.ldo + r;
        const bool vec = a.vec_out && r + 8 <= a.rows;
        const int cnt = (int)min((int64_t)8, a.rows - r);
        auto put = [&](uint16_t* out, u16x8 v) {
            if (vec) *reinterpret_cast<u16x8*>(out + o) = v;
            else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e < cnt) out[o + e] = v[e];
            }
        };
        u16x8 x;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = tile[rr + e][cc];
        if (!SCALE || a.o0) put(a.o0, x);
        if constexpr (SCALE) {
            u16x8 h, l, l2;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float v = bf2f(x[e]) * ts[rr + e];
                uint16_t hh, ll;
                split_bf16(v, hh, ll);
                h[e] = hh;
                l[e] = ll;
                // v - hi and then - lo are exact in float32 (each term keeps v's leading bits)
                l2[e] = f2bf((v - bf2f(hh)) - bf2f(ll));
            }
            put(a.hi, h);
            put(a.lo, l);
            put(a.lo2, l2);
        }
    }
}

static bool rows16(const void* p, int64_t ld) { return !p || (((uintptr_t)p & 15) == 0 && ld % 8 == 0); }

hipError_t transpose_u16(const uint16_t* in, int64_t ldi, uint16_t* out, int64_t ldo, int64_t rows, int64_t cols,
                         hipStream_t st) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const int64_t tr = (rows + 63) / 64, tc = (cols + 63) / 64;
    const TransposeArgs a{in, ldi, nullptr, out, nullptr, nullptr, nullptr, ldo, rows, cols, tc, rows16(in, ldi),
                          rows16(out, ldo)};
    hipLaunchKernelGGL(transpose_kernel<false>, dim3((unsigned)(tr * tc)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t transpose_scale_split(const uint16_t* in, int64_t ldi, const float* s, uint16_t* plain, uint16_t* hi,
                                 uint16_t* lo, uint16_t* lo2, int64_t ldo, int64_t rows, int64_t cols, hipStream_t st) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const int64_t tr = (rows + 63) / 64, tc = (cols + 63) / 64;
    const TransposeArgs a{in, ldi, s, plain, hi, lo, lo2, ldo, rows, cols, tc, rows16(in, ldi),
                          rows16(plain, ldo) && rows16(hi, ldo) && rows16(lo, ldo) && rows16(lo2, ldo)};
    hipLaunchKernelGGL(transpose_kernel<true>, dim3((unsigned)(tr * tc)), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------- sum of float32 product slices
// C[i][j] (+)= sum_z S[z][i - r0][j] in float64, z in order, for the rows [r0, r1); SYM: only the slices'
// lower tiles exist (a symmetric product; ncols = r1), and the values below the diagonal go to both
// sides of it, so the sum stays exactly symmetric.  One 32 x 32 tile per block (lower tiles only with
// SYM); bound by HBM.
template <bool SYM, class Out>
__global__ __launch_bounds__(256) void add_slices_kernel(const float* __restrict__ S, int64_t always, int64_t slices,
                                                         const int* __restrict__ flag, int64_t r0, int64_t r1,
                                                         int64_t ncols, int accumulate, Out* __restrict__ C,
                                                         int64_t ldc, int64_t tiles) {
    __shared__ double tile[32][33];
    if (flag && *flag == 0) slices = always;
    int64_t ti, tj;
    if constexpr (SYM) {
        const int64_t t0 = r0 / 32, b = t0 * (t0 + 1) / 2 + blockIdx.x;
        ti = (int64_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
        while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
        while (ti * (ti + 1) / 2 > b) --ti;
        tj = b - ti * (ti + 1) / 2;
    } else {
        ti = r0 / 32 + blockIdx.x / tiles;
        tj = blockIdx.x % tiles;
    }
    const int rr = threadIdx.x >> 3, cc = (threadIdx.x & 7) * 4;
    const int64_t i = ti * 32 + rr, j = tj * 32 + cc, stride = (r1 - r0) * ncols;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (i < r1) {
        const float* p = S + (i - r0) * ncols + j;
        if (ncols % 4 == 0 && j < ncols) {
#pragma unroll 4
            for (int64_t z = 0; z < slices; ++z) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(p + z * stride);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += (double)x[e];
            }
        } else {
            for (int64_t z = 0; z < slices; ++z)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (j + e < ncols) v[e] += (double)p[z * stride + e];
        }
    }
    // this thread's four values of row r from column c, and for a symmetric product those of the
    // mirrored tile: all old values are loaded before any is stored (C's loads cannot pass its stores)
    struct Four {
        Out* p;
        int n;
        double x[4], old[4];
    };
    auto four = [&](int64_t r, int64_t c, bool in, int64_t end) {
        Four q;
        q.p = C + r * ldc + c;
        q.n = in ? (int)max((int64_t)0, min((int64_t)4, end - c)) : 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) q.old[e] = accumulate && e < q.n ? (double)q.p[e] : 0.0;
        return q;
    };
    auto put = [&](const Four& q) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < q.n) q.p[e] = (Out)(accumulate ? q.old[e] + q.x[e] : q.x[e]);
    };
    Four own = four(i, j, i < r1, ncols);
    if constexpr (SYM) {
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[rr][cc + e] = v[e];
        const int64_t mi = tj * 32 + rr, mj = ti * 32 + cc;  // the mirrored tile's row and columns
        Four mirror = four(mi, mj, ti != tj && mi < ncols, r1);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) mirror.x[e] = tile[cc + e][rr];
        if (ti == tj) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (cc + e > rr) v[e] = tile[cc + e][rr];
        }
        put(mirror);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) own.x[e] = v[e];
    put(own);
}

template <class Out>
static hipError_t add_slices_t(const float* S, int64_t always, int64_t slices, const int* flag, int64_t r0, int64_t r1,
                               int64_t N, bool symmetric, bool accumulate, Out* C, int64_t ldc, hipStream_t st) {
    if (r1 <= r0 || N <= 0) return hipSuccess;
    const int64_t t0 = r0 / 32, t1 = (r1 + 31) / 32, tn = (N + 31) / 32;
    if (symmetric)
        hipLaunchKernelGGL((add_slices_kernel<true, Out>), dim3((unsigned)((t1 * (t1 + 1) - t0 * (t0 + 1)) / 2)),
                           dim3(256), 0, st, S, always, slices, flag, r0, r1, r1, (int)accumulate, C, ldc, tn);
    else
        hipLaunchKernelGGL((add_slices_kernel<false, Out>), dim3((unsigned)((t1 - t0) * tn)), dim3(256), 0, st, S,
                           always, slices, flag, r0, r1, N, (int)accumulate, C, ldc, tn);
    return hipGetLastError();
}
hipError_t add_slices(const float* S, int64_t always, int64_t slices, const int* flag, int64_t r0, int64_t r1,
                      int64_t N, bool symmetric, bool accumulate, double* C, int64_t ldc, hipStream_t st) {
    return add_slices_t(S, always, slices, flag, r0, r1, N, symmetric, accumulate, C, ldc, st);
}
hipError_t add_slices(const float* S, int64_t always, int64_t slices, const int* flag, int64_t r0, int64_t r1,
                      int64_t N, bool symmetric, bool accumulate, float* C, int64_t ldc, hipStream_t st) {
    return add_slices_t(S, always, slices, flag, r0, r1, N, symmetric, accumulate, C, ldc, st);
}

// Input perturbation of one token chunk, transposed: delta = Xhat - X (rows = tokens), and
// the hi/lo bf16 pairs of s[r] * delta and of delta, written as [cols][rows].
__global__ __launch_bounds__(256) void transpose_delta_kernel(const uint16_t* __restrict__ Xh,
                                                              const uint16_t* __restrict__ X, int64_t ldi,
                                                              const float* __restrict__ s, uint16_t* __restrict__ sdh,
                                                              uint16_t* __restrict__ sdl, uint16_t* __restrict__ dh,
                                                              uint16_t* __restrict__ dl, int64_t ldo, int64_t rows,
                                                              int64_t cols, int64_t tiles_c) {
    __shared__ float td[64][65];
    __shared__ float ts[64];
    const int64_t tr = blockIdx.x / tiles_c, tc = blockIdx.x % tiles_c;
    const int64_t r0 = tr * 64, c0 = tc * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int rr = ty; rr < 64; rr += 4) {
        const int64_t r = r0 + rr, c = c0 + tx;
        float v = 0.f;
        if (r < rows && c < cols) v = bf2f(Xh[r * ldi + c]) - bf2f(X[r * ldi + c]);
        td[rr][tx] = v;
    }
    if (threadIdx.x < 64) {
        const int64_t r = r0 + threadIdx.x;
        ts[threadIdx.x] = (s && r < rows) ? s[r] : 1.f;
    }
    __syncthreads();
    for (int cc = ty; cc < 64; cc += 4) {
        const int64_t c = c0 + cc, r = r0 + tx;
        if (r < rows && c < cols) {
            const float d = td[tx][cc];
            uint16_t hi, lo;
            split_bf16(d * ts[tx], hi, lo);
            sdh[c * ldo + r] = hi;
            sdl[c * ldo + r] = lo;
            split_bf16(d, hi, lo);
            dh[c * ldo + r] = hi;
            dl[c * ldo + r] = lo;
        }
    }
}

hipError_t transpose_delta_split(const uint16_t* Xh, const uint16_t* X, int64_t ldi, const float* s, uint16_t* sdh,
                                 uint16_t* sdl, uint16_t* dh, uint16_t* dl, int64_t ldo, int64_t rows, int64_t cols,
                                 hipStream_t st) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const int64_t tr = (rows + 63) / 64, tc = (cols + 63) / 64;
    hipLaunchKernelGGL(transpose_delta_kernel, dim3((unsigned)(tr * tc)), dim3(256), 0, st, Xh, X, ldi, s, sdh, sdl,
                       dh, dl, ldo, rows, cols, tc);
    return hipGetLastError();
}

// hi/lo bf16 pair of float(in[i][j]), rows of `cols` values written with stride ldo
__global__ void split_f64_kernel(const double* __restrict__ in, uint16_t* __restrict__ hi, uint16_t* __restrict__ lo,
                                 int64_t cols, int64_t ldo, int64_t total) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t o = (e / cols) * ldo + e % cols;
        uint16_t h, l;
        split_bf16((float)in[e], h, l);
        hi[o] = h;
        lo[o] = l;
    }
}

hipError_t split_f64(const double* in, uint16_t* hi, uint16_t* lo, int64_t ldo, int64_t rows, int64_t cols,
                     hipStream_t st) {
    const int64_t total = rows * cols;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_f64_kernel, dim3(grid_for(total, 4)), dim3(TB), 0, st, in, hi, lo, cols, ldo, total);
    return hipGetLastError();
}

// Row-wise kernels over activations: 8 columns a thread, a row to 2^row_log2 threads (all TB of them
// from 8 TB columns on), rows past the launch's in further rounds.  The outputs' rows are 16-byte
// aligned and padded to whole chunks of 8 columns (the padding is written, with zeros); inputs are
// loaded 16 bytes at a time where theirs are.
struct RowSpread {
    int64_t rows, cols;
    int row_log2, vec;
    unsigned grid;
};
static RowSpread row_spread(int64_t rows, int64_t cols, bool vec) {
    RowSpread r{rows, cols, 0, vec, 0};
    while ((1 << r.row_log2) < std::min<int64_t>((cols + 7) / 8, TB)) ++r.row_log2;
    const int64_t per = TB >> r.row_log2;
    // a launch holds less than 2^32 threads: 2^20 blocks at most, whatever the token count
    r.grid = (unsigned)std::min<int64_t>((rows + per - 1) / per, 1 << 20);
    return r;
}
// f(row, column) for this thread's chunks of 8 columns
template <class F>
__device__ __forceinline__ void each_chunk8(const RowSpread& r, const F& f) {
    const int per = TB >> r.row_log2, wide = 1 << r.row_log2;
    for (int64_t i = (int64_t)blockIdx.x * per + (threadIdx.x >> r.row_log2); i < r.rows; i += (int64_t)gridDim.x * per)
        for (int64_t j = (threadIdx.x & (wide - 1)) * 8; j < r.cols; j += wide * 8) f(i, j);
}
__device__ __forceinline__ u16x8 chunk8(const uint16_t* p, int64_t j, const RowSpread& r) {
    u16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
    if (r.vec && j + 8 <= r.cols) return *reinterpret_cast<const u16x8*>(p + j);
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (j + e < r.cols) v[e] = p[j + e];
    return v;
}

// Rows of `cols` bf16 values copied to stride ldo: activations whose rows are not a multiple of 16
// bytes, or whose tokens have places of their own, laid out once for the GEMMs' direct-to-LDS loads.
__global__ __launch_bounds__(TB) void place_rows_kernel(const uint16_t* __restrict__ in, int64_t ldi,
                                                        uint16_t* __restrict__ out, int64_t ldo, plan::Places L,
                                                        RowSpread r) {
    each_chunk8(r, [&](int64_t i, int64_t j) {
        const int64_t t = plan::token_at(L, i);
        const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
        *reinterpret_cast<u16x8*>(out + i * ldo + j) = t >= 0 ? chunk8(in + t * ldi, j, r) : zero;
    });
}

hipError_t place_rows_u16(const uint16_t* in, int64_t ldi, uint16_t* out, int64_t ldo, int64_t cols,
                          const plan::Places& L, hipStream_t st) {
    if (L.count <= 0 || cols <= 0) return hipSuccess;
    if (!rows16(out, ldo)) return hipErrorInvalidValue;
    const RowSpread r = row_spread(L.count, cols, rows16(in, ldi));
    hipLaunchKernelGGL(place_rows_kernel, dim3(r.grid), dim3(TB), 0, st, in, ldi, out, ldo, L, r);
    return hipGetLastError();
}

hipError_t copy_rows_u16(const uint16_t* in, int64_t ldi, uint16_t* out, int64_t ldo, int64_t rows, int64_t cols,
                         hipStream_t st) {
    return place_rows_u16(in, ldi, out, ldo, cols, plan::place_tokens(rows, rows, rows), st);
}

__global__ void place_f32_kernel(const float* __restrict__ in, float* __restrict__ out, plan::Places L) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < L.count; p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t t = plan::token_at(L, p);
        out[p] = t >= 0 ? in[t] : 0.f;
    }
}

hipError_t place_f32(const float* in, float* out, const plan::Places& L, hipStream_t st) {
    if (L.count <= 0) return hipSuccess;
    hipLaunchKernelGGL(place_f32_kernel, dim3(grid_for(L.count, 1)), dim3(TB), 0, st, in, out, L);
    return hipGetLastError();
}

__device__ __forceinline__ void split3(float x, uint16_t& h, uint16_t& l, uint16_t& l2) {
    h = f2bf(x);
    const float r1 = x - bf2f(h);
    l = f2bf(r1);
    l2 = f2bf(r1 - bf2f(l));
}

__global__ void split3_f64_kernel(const double* __restrict__ in, uint16_t* __restrict__ hi, uint16_t* __restrict__ lo,
                                  uint16_t* __restrict__ lo2, int64_t count) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x)
        split3((float)in[e], hi[e], lo[e], lo2[e]);
}

hipError_t split3_f64(const double* in, uint16_t* hi, uint16_t* lo, uint16_t* lo2, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(split3_f64_kernel, dim3(grid_for(count, 4)), dim3(TB), 0, st, in, hi, lo, lo2, count);
    return hipGetLastError();
}

// One wave's verdict on its lower terms: a plain store of 1, skipped once the flag is up (every
// writer stores the same value).
__device__ __forceinline__ void raise_flag(int* flag, bool any) {
    if (flag && __ballot(any) != 0 && (threadIdx.x & 63) == 0 && *(volatile int*)flag == 0) *(volatile int*)flag = 1;
}

// One row and 1024 columns per block, 4 columns per thread (16-byte loads, 8-byte stores where the
// rows allow them): bound by HBM (14 weight matrices of an 8B-shaped block: 77 -> 58 us on average
// against one element per thread and a 64-bit division each).
__global__ __launch_bounds__(256) void split3_f32_kernel(const float* __restrict__ A, int64_t lda,
                                                         uint16_t* __restrict__ hi, uint16_t* __restrict__ lo,
                                                         uint16_t* __restrict__ lo2, int64_t ld, int64_t cols,
                                                         int* __restrict__ flag, int vec) {
    typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
    const int64_t c = ((int64_t)blockIdx.y * 256 + threadIdx.x) * 4;
    const float* a = A + (int64_t)blockIdx.x * lda + c;
    const int64_t o = (int64_t)blockIdx.x * ld + c;
    uint32_t any = 0;
    if (vec && c + 4 <= cols) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(a);
        u16x4 h, l, l2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint16_t t0, t1, t2;
            split3(x[e], t0, t1, t2);
            h[e] = t0;
            l[e] = t1;
            l2[e] = t2;
            any |= (uint32_t)(t1 | t2) & 0x7FFFu;
        }
        *reinterpret_cast<u16x4*>(hi + o) = h;
        *reinterpret_cast<u16x4*>(lo + o) = l;
        *reinterpret_cast<u16x4*>(lo2 + o) = l2;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < cols) {
                split3(a[e], hi[o + e], lo[o + e], lo2[o + e]);
                any |= (uint32_t)(lo[o + e] | lo2[o + e]) & 0x7FFFu;
            }
    }
    raise_flag(flag, any != 0);
}

hipError_t split3_f32(const float* A, int64_t lda, uint16_t* hi, uint16_t* lo, uint16_t* lo2, int64_t ld,
                      int64_t rows, int64_t cols, int* flag, hipStream_t st) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    auto al = [](const void* p, uintptr_t b) { return ((uintptr_t)p & (b - 1)) == 0; };
    const int vec = al(A, 16) && lda % 4 == 0 && al(hi, 8) && al(lo, 8) && al(lo2, 8) && ld % 4 == 0;
    hipLaunchKernelGGL(split3_f32_kernel, dim3((unsigned)rows, (unsigned)((cols + 1023) / 1024)), dim3(256), 0, st, A,
                       lda, hi, lo, lo2, ld, cols, flag, vec);
    return hipGetLastError();
}

// Transposed terms of a float32 matrix through a 64 x 64 LDS tile: 16-byte loads along a row and
// 16-byte stores along a column where the arrays allow them; bound by HBM.
__global__ __launch_bounds__(256) void transpose_split3_f32_kernel(const float* __restrict__ in, int64_t ldi,
                                                                   uint16_t* __restrict__ hi, uint16_t* __restrict__ lo,
                                                                   uint16_t* __restrict__ lo2, int64_t ldo,
                                                                   int64_t rows, int64_t cols, int64_t tiles_c,
                                                                   int* __restrict__ flag, int vec_in, int vec_out) {
    __shared__ float tile[64][65];
    const int64_t r0 = (blockIdx.x / tiles_c) * 64, c0 = (blockIdx.x % tiles_c) * 64;
    const int t = threadIdx.x;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int rr = (t >> 4) + 16 * p, cc = (t & 15) * 4;
        const int64_t r = r0 + rr, c = c0 + cc;
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        if (r < rows) {
            const float* q = in + r * ldi + c;
            if (vec_in && c + 4 <= cols) x = *reinterpret_cast<const f32x4*>(q);
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + e < cols) x[e] = q[e];
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[rr][cc + e] = x[e];
    }
    __syncthreads();
    uint32_t any = 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int cc = (t >> 3) + 32 * p, rr = (t & 7) * 8;
        const int64_t c = c0 + cc, r = r0 + rr;
        if (c >= cols || r >= rows) continue;
        const int64_t o = c * ldo + r;
        u16x8 h, l, l2;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            uint16_t t0, t1, t2;
            split3(tile[rr + e][cc], t0, t1, t2);
            h[e] = t0;
            l[e] = t1;
            l2[e] = t2;
            any |= (uint32_t)(t1 | t2) & 0x7FFFu;  // rows past the end hold zeros
        }
        auto put = [&](uint16_t* out, u16x8 v) {
            if (vec_out && r + 8 <= rows) *reinterpret_cast<u16x8*>(out + o) = v;
            else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (r + e < rows) out[o + e] = v[e];
            }
        };
        put(hi, h);
        put(lo, l);
        if (lo2) put(lo2, l2);
    }
    raise_flag(flag, any != 0);
}

hipError_t transpose_split3_f32(const float* in, int64_t ldi, uint16_t* hi, uint16_t* lo, uint16_t* lo2, int64_t ldo,
                                int64_t rows, int64_t cols, int* flag, hipStream_t st) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const int64_t tr = (rows + 63) / 64, tc = (cols + 63) / 64;
    const int vec_in = ((uintptr_t)in & 15) == 0 && ldi % 4 == 0;
    const int vec_out = rows16(hi, ldo) && rows16(lo, ldo) && rows16(lo2, ldo);
    hipLaunchKernelGGL(transpose_split3_f32_kernel, dim3((unsigned)(tr * tc)), dim3(256), 0, st, in, ldi, hi, lo, lo2,
                       ldo, rows, cols, tc, flag, vec_in, vec_out);
    return hipGetLastError();
}

// flag |= 1 when any of the count bf16 values is nonzero (either sign of zero counts as zero)
__global__ void any_nonzero_u16_kernel(const uint16_t* __restrict__ p, int64_t count, int* __restrict__ flag) {
    uint32_t any = 0;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x)
        any |= p[e] & 0x7FFFu;
    if (any) atomicOr(flag, 1);
}

hipError_t any_nonzero_u16(const uint16_t* p, int64_t count, int* flag, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(any_nonzero_u16_kernel, dim3(grid_for(count, 8)), dim3(TB), 0, st, p, count, flag);
    return hipGetLastError();
}

// G[i][j] = C0[i][c1 + j] + P[i][c1 + j]   (m x w, C0 and P with row stride ld)
__global__ void gram_grad_kernel(const float* __restrict__ C0, const float* __restrict__ P, int64_t ld, int64_t c1,
                                 int64_t w, int64_t total, float* __restrict__ G) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / w, j = c1 + e % w;
        G[e] = C0[i * ld + j] + P[i * ld + j];
    }
}

hipError_t gram_grad(const float* C0, const float* P, int64_t ld, int64_t c1, int64_t m, int64_t w, float* G,
                     hipStream_t st) {
    const int64_t total = m * w;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(gram_grad_kernel, dim3(grid_for(total, 4)), dim3(TB), 0, st, C0, P, ld, c1, w, total, G);
    return hipGetLastError();
}

// out = A - double(B) (float64 minus float32, elementwise)
__global__ void sub_f64_f32_kernel(const double* __restrict__ A, const float* __restrict__ B, double* __restrict__ out,
                                   int64_t count) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x)
        out[e] = A[e] - (double)B[e];
}

hipError_t sub_f64_f32(const double* A, const float* B, double* out, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(sub_f64_f32_kernel, dim3(grid_for(count, 4)), dim3(TB), 0, st, A, B, out, count);
    return hipGetLastError();
}

// Deterministic dot product of two float64 arrays: each of DOT_BLOCKS blocks sums a fixed
// strided subset in a fixed order and reduces it in a fixed tree; partials[b] receives it.
constexpr int DOT_BLOCKS = 1024;
__global__ __launch_bounds__(256) void dot_f64_kernel(const double* __restrict__ X, const double* __restrict__ Y,
                                                      int64_t count, double* __restrict__ partials) {
    __shared__ double red[256];
    double acc = 0.0;
    for (int64_t e = blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)DOT_BLOCKS * 256) acc += X[e] * Y[e];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[blockIdx.x] = red[0];
}

// Gram form of a BGD step: sum over all weights of (2 C0 + P) (W - W0), same fixed-order
// partials as dot_f64.
__global__ __launch_bounds__(256) void dot_gram_kernel(const float* __restrict__ C0, const float* __restrict__ P,
                                                       const double* __restrict__ W, const float* __restrict__ W0,
                                                       int64_t count, double* __restrict__ partials) {
    __shared__ double red[256];
    double acc = 0.0;
    for (int64_t e = blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)DOT_BLOCKS * 256)
        acc += (2.0 * (double)C0[e] + (double)P[e]) * (W[e] - (double)W0[e]);
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[blockIdx.x] = red[0];
}

hipError_t dot_gram(const float* C0, const float* P, const double* W, const float* W0, int64_t count,
                    double* partials, hipStream_t st) {
    hipLaunchKernelGGL(dot_gram_kernel, dim3(DOT_BLOCKS), dim3(256), 0, st, C0, P, W, W0, count, partials);
    return hipGetLastError();
}

hipError_t dot_f64(const double* X, const double* Y, int64_t count, double* partials, hipStream_t st) {
    hipLaunchKernelGGL(dot_f64_kernel, dim3(DOT_BLOCKS), dim3(256), 0, st, X, Y, count, partials);
    return hipGetLastError();
}
int64_t dot_f64_partials() { return DOT_BLOCKS; }

// ---------------------------------------------------------------- splits
__global__ void split_diff_f32_kernel(const float* __restrict__ A, int64_t lda, const float* __restrict__ Bm,
                                      int64_t ldb, uint16_t* __restrict__ hi, uint16_t* __restrict__ lo, int64_t ld,
                                      int64_t rows, int64_t cols) {
    const int64_t total = rows * cols;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        int64_t i = e / cols, j = e % cols;
        float v = A[i * lda + j];
        if (Bm) v -= Bm[i * ldb + j];
        uint16_t h, l;
        split_bf16(v, h, l);
        hi[i * ld + j] = h;
        lo[i * ld + j] = l;
    }
}

__global__ void split_diff_f64_kernel(const double* __restrict__ A, int64_t lda, const float* __restrict__ Bm,
                                      int64_t ldb, uint16_t* __restrict__ hi, uint16_t* __restrict__ lo, int64_t ld,
                                      int64_t rows, int64_t cols) {
    const int64_t total = rows * cols;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / cols, j = e % cols;
        const float v = (float)(A[i * lda + j] - (double)Bm[i * ldb + j]);
        uint16_t h, l;
        split_bf16(v, h, l);
        hi[i * ld + j] = h;
        lo[i * ld + j] = l;
    }
}

hipError_t split_diff_f64(const double* A, int64_t lda, const float* Bm, int64_t ldb, uint16_t* hi, uint16_t* lo,
                          int64_t ld, int64_t rows, int64_t cols, hipStream_t st) {
    const int64_t total = rows * cols;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_diff_f64_kernel, dim3(grid_for(total, 4)), dim3(TB), 0, st, A, lda, Bm, ldb, hi, lo, ld,
                       rows, cols);
    return hipGetLastError();
}

__global__ void widen_kernel(const float* __restrict__ in, double* __restrict__ out, int64_t count) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x)
        out[e] = (double)in[e];
}

__global__ void narrow_kernel(const double* __restrict__ in, float* __restrict__ out, int64_t count) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x)
        out[e] = (float)in[e];
}

hipError_t widen_f32(const float* in, double* out, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(widen_kernel, dim3(grid_for(count, 4)), dim3(TB), 0, st, in, out, count);
    return hipGetLastError();
}

hipError_t narrow_f64(const double* in, float* out, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(narrow_kernel, dim3(grid_for(count, 4)), dim3(TB), 0, st, in, out, count);
    return hipGetLastError();
}

hipError_t split_diff_f32(const float* A, int64_t lda, const float* Bm, int64_t ldb, uint16_t* hi, uint16_t* lo,
                          int64_t ld, int64_t rows, int64_t cols, hipStream_t st) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_diff_f32_kernel, dim3(grid_for(rows * cols, 4)), dim3(TB), 0, st, A, lda, Bm, ldb, hi, lo,
                       ld, rows, cols);
    return hipGetLastError();
}

// Blended metric of Eq. slide_window as a bf16 pair: x = alpha (M or I)[i][k] + (1 - alpha) P[i][k]
// (P may be NULL), hi = bf16(x), lo = bf16(x - hi); m x m, written with row stride ldo.
__global__ void blend_split_kernel(const float* __restrict__ M, const float* __restrict__ P, float alpha, int64_t m,
                                   uint16_t* __restrict__ hi, uint16_t* __restrict__ lo, int64_t ldo) {
    const int64_t total = m * m;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / m, k = e % m;
        float v = alpha * (M ? M[e] : (i == k ? 1.f : 0.f));
        if (P) v += (1.f - alpha) * P[e];
        uint16_t h, l;
        split_bf16(v, h, l);
        hi[i * ldo + k] = h;
        lo[i * ldo + k] = l;
    }
}

hipError_t blend_split(const float* M, const float* P, float alpha, int64_t m, uint16_t* hi, uint16_t* lo, int64_t ldo,
                       hipStream_t st) {
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(blend_split_kernel, dim3(grid_for(m * m, 4)), dim3(TB), 0, st, M, P, alpha, m, hi, lo, ldo);
    return hipGetLastError();
}

__global__ __launch_bounds__(TB) void split_diff_bf16_kernel(const uint16_t* __restrict__ a,
                                                             const uint16_t* __restrict__ b, uint16_t* __restrict__ hi,
                                                             uint16_t* __restrict__ lo, int64_t ldo, plan::Places L,
                                                             int64_t p0, RowSpread r) {
    each_chunk8(r, [&](int64_t i, int64_t j) {
        const int64_t t = plan::token_at(L, p0 + i);
        u16x8 x = {0, 0, 0, 0, 0, 0, 0, 0}, y = x, h, l;
        if (t >= 0) {
            x = chunk8(a + t * r.cols, j, r);
            y = chunk8(b + t * r.cols, j, r);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            uint16_t hh, ll;
            split_bf16(bf2f(x[e]) - bf2f(y[e]), hh, ll);  // exact in float32 for bf16 inputs of similar magnitude
            h[e] = hh;
            l[e] = ll;
        }
        *reinterpret_cast<u16x8*>(hi + i * ldo + j) = h;
        *reinterpret_cast<u16x8*>(lo + i * ldo + j) = l;
    });
}

hipError_t split_diff_bf16(const uint16_t* a, const uint16_t* b, uint16_t* hi, uint16_t* lo, int64_t ldo, int64_t rows,
                           int64_t cols, const plan::Places& L, int64_t p0, hipStream_t st) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    if (!rows16(hi, ldo) || !rows16(lo, ldo)) return hipErrorInvalidValue;
    const RowSpread r = row_spread(rows, cols, rows16(a, cols) && rows16(b, cols));
    hipLaunchKernelGGL(split_diff_bf16_kernel, dim3(r.grid), dim3(TB), 0, st, a, b, hi, lo, ldo, L, p0, r);
    return hipGetLastError();
}

// ---------------------------------------------------------------- deterministic reduction
__global__ __launch_bounds__(256) void reduce_partials_kernel(const double* __restrict__ p, int64_t count,
                                                              double scale, double* out) {
    __shared__ double red[256];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += 256) acc += p[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0] * scale;
}

hipError_t reduce_partials(const double* partials, int64_t count, double scale, double* out, hipStream_t st) {
    hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(256), 0, st, partials, count, scale, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- split-K reduction + Adam
// Bias-corrected Adam in the Kingma-Ba form: m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// w -= lr * (m * bc1) / (sqrt(v * bc2) + eps).  The moments and the step are float32; the
// step is added to the float64 working weight.
__device__ __forceinline__ void adam_elem(const AdamArgs& a, int64_t i, int64_t j, float g) {
    const int64_t idx = i * a.n + j;
    float mv = a.beta1 * a.mA[idx] + (1.f - a.beta1) * g;
    float vv = a.beta2 * a.vA[idx] + (1.f - a.beta2) * g * g;
    a.mA[idx] = mv;
    a.vA[idx] = vv;
    float mh = mv * a.bc1;
    float vh = vv * a.bc2;
    const float step = a.lr * mh / (sqrtf(vh) + a.eps);
    const double w = a.W[idx] - (double)step;
    a.W[idx] = w;
    const int64_t di = i * a.ldd + j;
    if (a.Dacc) {
        const float d = (a.inc_reset ? 0.f : a.Dacc[idx]) - step;
        a.Dacc[idx] = d;
        a.Dinc[di] = f2bf(d);
    }
    if (!a.Dhi) return;
    uint16_t h, l;
    split_bf16((float)(w - (double)a.W0[idx]), h, l);
    a.Dhi[di] = h;
    a.Dlo[di] = l;
}

__global__ void adam_kernel(AdamArgs a) {
    const int64_t w = a.n - a.c1;
    const int64_t total = a.m * w;
    const int64_t zstride = a.m * w;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        float g = 0.f;
        for (int64_t z = 0; z < a.splits; ++z) g += a.Gp[z * zstride + e];
        if (a.g0_mode == 2) g += a.G0[e];
        else if (a.g0_mode == 1) a.G0[e] = g;
        g *= a.gscale;
        int64_t i = e / w, j = a.c1 + e % w;
        adam_elem(a, i, j, g);
    }
}

hipError_t adam_update(const AdamArgs& a, hipStream_t st) {
    const int64_t total = a.m * (a.n - a.c1);
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(adam_kernel, dim3(grid_for(total, 4)), dim3(TB), 0, st, a);
    return hipGetLastError();
}

// The cross term <G0, Dinc> in fixed-order per-block float64 sums, then one block adds it to L0
// and the partial sums of s_t acc^2.
constexpr int INC_DOT_BLOCKS = 512;
__global__ __launch_bounds__(256) void inc_dot_kernel(const float* __restrict__ G0, const uint16_t* __restrict__ Dinc,
                                                      int64_t ldd, int64_t m, int64_t w, double* __restrict__ dots) {
    __shared__ double red[256];
    double acc = 0.0;
    for (int64_t i = blockIdx.x; i < m; i += INC_DOT_BLOCKS) {  // rows, coalesced along each
        const float* g = G0 + i * w;
        const uint16_t* d = Dinc + i * ldd;
        for (int64_t j = threadIdx.x; j < w; j += 256) acc += (double)g[j] * (double)bf2f(d[j]);
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) dots[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void inc_loss_kernel(const double* __restrict__ L0, const double* __restrict__ dots,
                                                       const double* __restrict__ parts, int64_t nparts, double T,
                                                       double* __restrict__ out) {
    __shared__ double rd[256], rp[256];
    double d = 0.0, p = 0.0;
    for (int64_t k = threadIdx.x; k < INC_DOT_BLOCKS; k += 256) d += dots[k];
    for (int64_t k = threadIdx.x; k < nparts; k += 256) p += parts[k];
    rd[threadIdx.x] = d;
    rp[threadIdx.x] = p;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) {
            rd[threadIdx.x] += rd[threadIdx.x + k];
            rp[threadIdx.x] += rp[threadIdx.x + k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = *L0 + rd[0] / T + 0.5 / T * rp[0];
}

int64_t inc_loss_partials() { return INC_DOT_BLOCKS; }

hipError_t inc_loss(const double* L0, const float* G0, const uint16_t* Dinc, int64_t ldd, int64_t m, int64_t w,
                    const double* parts, int64_t nparts, double T, double* dots, double* out, hipStream_t st) {
    hipLaunchKernelGGL(inc_dot_kernel, dim3(INC_DOT_BLOCKS), dim3(256), 0, st, G0, Dinc, ldd, m, w, dots);
    hipLaunchKernelGGL(inc_loss_kernel, dim3(1), dim3(256), 0, st, L0, dots, parts, nparts, T, out);
    return hipGetLastError();
}

__global__ void adam_dense_kernel(AdamArgs a, const float* __restrict__ G) {
    const int64_t w = a.n - a.c1;
    const int64_t total = a.m * w;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        int64_t i = e / w, j = a.c1 + e % w;
        adam_elem(a, i, j, G[e]);
    }
}

hipError_t adam_update_dense(const AdamArgs& a, const float* G, hipStream_t st) {
    const int64_t total = a.m * (a.n - a.c1);
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(adam_dense_kernel, dim3(grid_for(total, 4)), dim3(TB), 0, st, a, G);
    return hipGetLastError();
}

__global__ void reduce_splits_kernel(const float* __restrict__ Gp, int64_t splits, int64_t total, float gscale,
                                     float* __restrict__ G, int accumulate) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        float g = 0.f;
        for (int64_t z = 0; z < splits; ++z) g += Gp[z * total + e];
        g *= gscale;
        G[e] = accumulate ? G[e] + g : g;
    }
}

hipError_t reduce_splits(const float* Gp, int64_t splits, int64_t m, int64_t w, float gscale, float* G,
                         bool accumulate, hipStream_t st) {
    const int64_t total = m * w;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(reduce_splits_kernel, dim3(grid_for(total, 4)), dim3(TB), 0, st, Gp, splits, total, gscale, G,
                       (int)accumulate);
    return hipGetLastError();
}

}  // namespace realq
