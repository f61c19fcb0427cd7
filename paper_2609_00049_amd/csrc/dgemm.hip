// Float64 GEMM, all row-major: the products of the final loss with a dense metric, written through
// the calibration Gram matrices, of the Gram form's start and of the pulled-back metric of small modules.
#include "common.h"
#include "f64mma.h"
#include "kernels.h"

namespace realq {

// C = A B or C += A B in float64 on the matrix cores, any sizes and strides; 128 x 128 tiles once
// they fill the chip, 64 x 64 below (four times as many workgroups).  Bound by the staging into LDS,
// whose loads are in flight during one K step only; 1000 x 1352 x 1352: 294 us on the vector units
// with 4 x 4 tiles, 113 us here.
// A_KC: A(i, k) = A[i * lda + k], else A[k * lda + i]; float32 operands enter exactly.
template <int T, bool A_KC, class EA, class EB, class Out>
__global__ __launch_bounds__(256, 2) void dgemm_kernel(const EA* __restrict__ A, int64_t lda,
                                                       const EB* __restrict__ B, int64_t ldb, Out* __restrict__ C,
                                                       int64_t ldc, int64_t M, int64_t N, int64_t K, int accumulate,
                                                       int64_t tiles_n, int vec_a, int vec_b) {
    using F = F64Tile<T>;
    __shared__ __attribute__((aligned(16))) double lds[4 * F::LDS];
    const int64_t m0 = (blockIdx.x / tiles_n) * T, n0 = (blockIdx.x % tiles_n) * T;
    f64x4 acc[F::SUB][F::SUB];
    const F64CheckOC<EB> b{B + n0, ldb, N - n0, K, vec_b != 0};
    if constexpr (A_KC)
        F::template product<true, false>(acc, lds, 0, K, F64CheckKC<EA>{A + m0 * lda, lda, M - m0, K, vec_a != 0}, b);
    else
        F::template product<false, false>(acc, lds, 0, K, F64CheckOC<EA>{A + m0, lda, M - m0, K, vec_a != 0}, b);
    F::each(acc, [&](int r, int c, double x) {
        const int64_t i = m0 + r, j = n0 + c;
        if (i >= M || j >= N) return;
        Out* p = C + i * ldc + j;
        *p = (Out)(accumulate ? (double)*p + x : x);
    });
}

template <int T, bool A_KC, class EA, class EB, class Out>
static hipError_t dgemm_tiles(const EA* A, int64_t lda, const EB* B, int64_t ldb, Out* C, int64_t ldc, int64_t M,
                              int64_t N, int64_t K, bool accumulate, hipStream_t st) {
    auto rows16 = [](const void* p, int64_t ld, int size) { return ((uintptr_t)p & 15) == 0 && ld % (16 / size) == 0; };
    const int64_t tm = (M + T - 1) / T, tn = (N + T - 1) / T;
    hipLaunchKernelGGL((dgemm_kernel<T, A_KC, EA, EB, Out>), dim3((unsigned)(tm * tn)), dim3(256), 0, st, A, lda, B, ldb,
                       C, ldc, M, N, K, (int)accumulate, tn, (int)rows16(A, lda, sizeof(EA)),
                       (int)rows16(B, ldb, sizeof(EB)));
    return hipGetLastError();
}

// P = W^T R or P += W^T R in float64 with R = Mn W (T1, [m_next, m] float64 work) or W; two launches or
// one of 64 x 64 tiles.  Bound by latency below one round of tiles: a K step of 16 takes about 1.5 us.
// plan::pullback_small says where, with both sides measured.
hipError_t pullback_f64(const float* W, const float* Mn, int64_t m_next, int64_t m, double* T1, bool accumulate,
                        float* P, hipStream_t st) {
    if (m_next <= 0 || m <= 0) return hipSuccess;
    if (!Mn) return dgemm_tiles<64, false>(W, m, W, m, P, m, m, m, m_next, accumulate, st);
    const hipError_t e = dgemm_tiles<64, true>(Mn, m_next, W, m, T1, m, m_next, m, m_next, false, st);
    return e != hipSuccess ? e : dgemm_tiles<64, false>(W, m, (const double*)T1, m, P, m, m, m, m_next, accumulate, st);
}

hipError_t dgemm(const double* A, int64_t lda, const double* B, int64_t ldb, double* C, int64_t ldc, int64_t M,
                 int64_t N, int64_t K, bool accumulate, hipStream_t st) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if ((M + 127) / 128 * ((N + 127) / 128) >= 256)
        return dgemm_tiles<128, true>(A, lda, B, ldb, C, ldc, M, N, K, accumulate, st);
    return dgemm_tiles<64, true>(A, lda, B, ldb, C, ldc, M, N, K, accumulate, st);
}

}  // namespace realq
