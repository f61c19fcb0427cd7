// Float64 GEMM, all row-major: the products of the final loss with a dense metric, written through
// the calibration Gram matrices, and of the Gram form's start.
#include "common.h"
#include "f64mma.h"
#include "kernels.h"

namespace realq {

// C = A B or C += A B in float64 on the matrix cores, any sizes and strides; 128 x 128 tiles once
// they fill the chip, 64 x 64 below (four times as many workgroups).  Bound by the staging into LDS,
// whose loads are in flight during one K step only; 1000 x 1352 x 1352: 294 us on the vector units
// with 4 x 4 tiles, 113 us here.
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

}  // namespace realq
