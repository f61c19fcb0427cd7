// GEMMs outside the bf16 pipeline, all row-major.
//   sgemm  C = beta*C + alpha*A*B in float32 (VALU, 64x64 output tile per 256-thread block, 4x4 per
//          thread, K staged through LDS): the window partner W_next^T M_next W_next (Eq.
//          slide_window).
//   dgemm  C (+)= A*B in float64 (matrix cores, f64mma.h): the products of the final loss with a
//          dense metric, written through the calibration Gram matrices.
#include "common.h"
#include "f64mma.h"
#include "kernels.h"

namespace realq {

namespace {
constexpr int TM = 64, TN = 64, TK = 16;
}

__global__ __launch_bounds__(256) void sgemm_kernel(SgemmArgs a, int64_t tiles_n) {
    __shared__ float sA[TK][TM + 4];
    __shared__ float sB[TK][TN + 4];
    const int64_t tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
    const int64_t m0 = tm * TM, n0 = tn * TN;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;  // 16 x 16 threads, 4x4 each
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

    for (int64_t k0 = 0; k0 < a.K; k0 += TK) {
        // A tile: 64 rows x 16 k -> 1024 values, 4 per thread
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int e = threadIdx.x + r * 256;
            int row = e / TK, kk = e % TK;
            int64_t gi = m0 + row, gk = k0 + kk;
            sA[kk][row] = (gi < a.M && gk < a.K) ? a.A[gi * a.lda + gk] : 0.f;
        }
        // B tile: 16 k x 64 cols
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int e = threadIdx.x + r * 256;
            int kk = e / TN, col = e % TN;
            int64_t gk = k0 + kk, gj = n0 + col;
            sB[kk][col] = (gk < a.K && gj < a.N) ? a.B[gk * a.ldb + gj] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < TK; ++kk) {
            float av[4], bv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i] = sA[kk][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) bv[j] = sB[kk][tx + 16 * j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int64_t gi = m0 + ty * 4 + i;
        if (gi >= a.M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int64_t gj = n0 + tx + 16 * j;
            if (gj >= a.N) continue;
            float* c = a.C + gi * a.ldc + gj;
            float v = a.alpha * acc[i][j];
            if (a.beta != 0.f) v = fmaf(a.beta, *c, v);
            *c = v;
        }
    }
}

// C = A B or C += A B in float64 on the matrix cores, any sizes and strides; 128 x 128 tiles once
// they fill the chip, 64 x 64 below (four times as many workgroups).
template <int T>
__global__ __launch_bounds__(256, 2) void dgemm_kernel(const double* __restrict__ A, int64_t lda,
                                                       const double* __restrict__ B, int64_t ldb,
                                                       double* __restrict__ C, int64_t ldc, int64_t M, int64_t N,
                                                       int64_t K, int accumulate, int64_t tiles_n, int vec_a,
                                                       int vec_b) {
    using F = F64Tile<T>;
    __shared__ __attribute__((aligned(16))) double lds[4 * F::LDS];
    const int64_t m0 = (blockIdx.x / tiles_n) * T, n0 = (blockIdx.x % tiles_n) * T;
    f64x4 acc[F::SUB][F::SUB];
    F::template product<true, false>(acc, lds, 0, K, F64CheckKC<double>{A + m0 * lda, lda, M - m0, K, vec_a != 0},
                                     F64CheckOC<double>{B + n0, ldb, N - n0, K, vec_b != 0});
    F::each(acc, [&](int r, int c, double x) {
        const int64_t i = m0 + r, j = n0 + c;
        if (i >= M || j >= N) return;
        double* p = C + i * ldc + j;
        *p = accumulate ? *p + x : x;
    });
}

hipError_t dgemm(const double* A, int64_t lda, const double* B, int64_t ldb, double* C, int64_t ldc, int64_t M,
                 int64_t N, int64_t K, bool accumulate, hipStream_t st) {
    if (M <= 0 || N <= 0) return hipSuccess;
    const int vec_a = ((uintptr_t)A & 15) == 0 && lda % 2 == 0, vec_b = ((uintptr_t)B & 15) == 0 && ldb % 2 == 0;
    const int64_t m128 = (M + 127) / 128, n128 = (N + 127) / 128, m64 = (M + 63) / 64, n64 = (N + 63) / 64;
    if (m128 * n128 >= 256)
        hipLaunchKernelGGL(dgemm_kernel<128>, dim3((unsigned)(m128 * n128)), dim3(256), 0, st, A, lda, B, ldb, C, ldc,
                           M, N, K, (int)accumulate, n128, vec_a, vec_b);
    else
        hipLaunchKernelGGL(dgemm_kernel<64>, dim3((unsigned)(m64 * n64)), dim3(256), 0, st, A, lda, B, ldb, C, ldc, M,
                           N, K, (int)accumulate, n64, vec_a, vec_b);
    return hipGetLastError();
}

hipError_t sgemm(const SgemmArgs& a, hipStream_t st) {
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    int64_t tiles_m = (a.M + TM - 1) / TM, tiles_n = (a.N + TN - 1) / TN;
    hipLaunchKernelGGL(sgemm_kernel, dim3((unsigned)(tiles_m * tiles_n)), dim3(256), 0, st, a, tiles_n);
    return hipGetLastError();
}

}  // namespace realq
