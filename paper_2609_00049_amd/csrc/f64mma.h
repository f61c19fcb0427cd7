// Float64 tile products on the matrix cores (v_mfma_f64_16x16x4_f64): the building block of the
// Cholesky factorisation, its triangular inverse, the trailing compensation update and the float64
// products of the dense-metric loss.
//
// A workgroup of 4 waves (2 x 2) forms a T x T tile of sum_k A(i, k) B(k, j), T = 64 or 128, K in
// slices of 16 through two LDS buffers.  The float64 matrix rate equals the vector rate on gfx950
// (about 72 TFLOP/s sustained), but a 16 x 16 x 4 product takes two 8-byte LDS reads per lane for
// 2048 FLOP where a 4 x 4 register tile of vector FMAs takes eight for the same work per k: the
// vector kernels these products replace were bound by LDS reads at 13 to 20 TFLOP/s.
//
// Element layouts of the instruction: A lane l holds (row l % 16, k l / 16), B lane l (k l / 16,
// column l % 16), the accumulator's element v of lane l is (row 4 v + l / 16, column l % 16).
#pragma once
#include "common.h"

namespace realq {

constexpr int F64_KS = 16;

template <int T>
struct F64Tile {
    // padded so that two adjacent k rows fall on different halves of the 64 banks
    static constexpr int SP = T + 16;
    static constexpr int SUB = T / 32;        // 16-wide sub-tiles per wave and dimension
    static constexpr int PASS = T / 64;       // 4-value loads per thread and slice
    static constexpr int LDS = F64_KS * SP;   // doubles of one operand slice

    // position of (k, o) in an operand slice; the XOR spreads the stores of operands that are
    // loaded along k over the banks and permutes reads (one k / 4 per instruction) harmlessly
    __device__ static __forceinline__ int at(int k, int o) { return k * SP + (o ^ (((k >> 2) & 3) << 3)); }

    // The 4 values a thread brings of slice k0.. in load pass p: along k (KC: value q at k + q, one
    // outer index) or along the outer index (value q at o + q, one k).
    template <bool KC>
    __device__ static __forceinline__ void where(int p, int& o, int& k) {
        const int t = threadIdx.x;
        if constexpr (KC) {
            o = (t >> 2) + 64 * p;
            k = (t & 3) * 4;
        } else {
            o = (t % (T / 4)) * 4;
            k = t / (T / 4) + (F64_KS / PASS) * p;
        }
    }
    template <bool KC, class F>
    __device__ static __forceinline__ void load(double (&r)[PASS][4], int64_t k0, const F& f) {
#pragma unroll
        for (int p = 0; p < PASS; ++p) {
            int o, k;
            where<KC>(p, o, k);
            f(o, k0 + k, r[p]);
        }
    }
    template <bool KC>
    __device__ static __forceinline__ void store(double* s, const double (&r)[PASS][4]) {
#pragma unroll
        for (int p = 0; p < PASS; ++p) {
            int o, k;
            where<KC>(p, o, k);
            if constexpr (KC) {
#pragma unroll
                for (int q = 0; q < 4; ++q) s[at(k + q, o)] = r[p][q];
            } else {
                double2* d = reinterpret_cast<double2*>(s + at(k, o));
                d[0] = make_double2(r[p][0], r[p][1]);
                d[1] = make_double2(r[p][2], r[p][3]);
            }
        }
    }
    __device__ static __forceinline__ void mfma(f64x4 (&acc)[SUB][SUB], const double* sa, const double* sb) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int ro = (wave >> 1) * (T / 2) + (lane & 15), co = (wave & 1) * (T / 2) + (lane & 15);
#pragma unroll
        for (int q = 0; q < F64_KS / 4; ++q) {
            double a[SUB], b[SUB];
#pragma unroll
            for (int i = 0; i < SUB; ++i) a[i] = sa[at(4 * q + (lane >> 4), ro + 16 * i)];
#pragma unroll
            for (int j = 0; j < SUB; ++j) b[j] = sb[at(4 * q + (lane >> 4), co + 16 * j)];
#pragma unroll
            for (int i = 0; i < SUB; ++i)
#pragma unroll
                for (int j = 0; j < SUB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
    // acc = sum over k in [k_lo, k_hi) (a whole number of slices, or the loaders return 0 past the
    // end).  la(o, k, r) and lb(o, k, r) fill r with 4 operand values as `where` describes.
    template <bool A_KC, bool B_KC, class LA, class LB>
    __device__ static __forceinline__ void product(f64x4 (&acc)[SUB][SUB], double* lds, int64_t k_lo, int64_t k_hi,
                                                   const LA& la, const LB& lb) {
#pragma unroll
        for (int i = 0; i < SUB; ++i)
#pragma unroll
            for (int j = 0; j < SUB; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
        if (k_lo >= k_hi) return;
        double ra[PASS][4], rb[PASS][4];
        load<A_KC>(ra, k_lo, la);
        load<B_KC>(rb, k_lo, lb);
        store<A_KC>(lds, ra);
        store<B_KC>(lds + 2 * LDS, rb);
        __syncthreads();
        int cur = 0;
        for (int64_t k = k_lo; k < k_hi; k += F64_KS) {
            const bool more = k + F64_KS < k_hi;
            if (more) {
                load<A_KC>(ra, k + F64_KS, la);
                load<B_KC>(rb, k + F64_KS, lb);
            }
            mfma(acc, lds + cur * LDS, lds + (2 + cur) * LDS);
            if (more) {
                store<A_KC>(lds + (cur ^ 1) * LDS, ra);
                store<B_KC>(lds + (2 + (cur ^ 1)) * LDS, rb);
            }
            __syncthreads();
            cur ^= 1;
        }
    }
    // f(row, column, value) for every element this lane holds
    template <class F>
    __device__ static __forceinline__ void each(const f64x4 (&acc)[SUB][SUB], const F& f) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int i = 0; i < SUB; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int j = 0; j < SUB; ++j)
                    f((wave >> 1) * (T / 2) + 16 * i + 4 * v + (lane >> 4), (wave & 1) * (T / 2) + 16 * j + (lane & 15),
                      acc[i][j][v]);
    }
};

// Loaders for operands of whole 64-blocks (dimensions and strides multiples of 64, 16-byte aligned).
// Outer indices past `lim` are clamped (their products are not stored).
struct F64LoadKC {  // element (o, k) at p[o * ld + k]
    const double* p;
    int64_t ld;
    int lim;
    __device__ __forceinline__ void operator()(int o, int64_t k, double (&r)[4]) const {
        o = o < lim ? o : lim - 1;
        const double2* q = reinterpret_cast<const double2*>(p + (int64_t)o * ld + k);
        const double2 u = q[0], v = q[1];
        r[0] = u.x; r[1] = u.y; r[2] = v.x; r[3] = v.y;
    }
};
struct F64LoadOC {  // element (o, k) at p[k * ld + o]
    const double* p;
    int64_t ld;
    int lim;
    __device__ __forceinline__ void operator()(int o, int64_t k, double (&r)[4]) const {
        o = o + 3 < lim ? o : lim - 4;
        const double2* q = reinterpret_cast<const double2*>(p + k * ld + o);
        const double2 u = q[0], v = q[1];
        r[0] = u.x; r[1] = u.y; r[2] = v.x; r[3] = v.y;
    }
};

// Loaders for any sizes, strides and alignment: zero outside [0, lim) x [0, K).
template <class E>
struct F64CheckKC {  // element (o, k) at p[o * ld + k]
    const E* p;
    int64_t ld, lim, K;
    bool vec;  // rows 16-byte aligned
    __device__ __forceinline__ void operator()(int o, int64_t k, double (&r)[4]) const {
        const E* q = p + (int64_t)o * ld + k;
        if (vec && o < lim && k + 3 < K) {
#pragma unroll
            for (int e = 0; e < 4; e += 16 / (int)sizeof(E)) {
                typedef E V __attribute__((ext_vector_type(16 / sizeof(E))));
                const V v = *reinterpret_cast<const V*>(q + e);
#pragma unroll
                for (int u = 0; u < 16 / (int)sizeof(E); ++u) r[e + u] = (double)v[u];
            }
            return;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (o < lim && k + e < K) ? (double)q[e] : 0.0;
    }
};
template <class E>
struct F64CheckOC {  // element (o, k) at p[k * ld + o]
    const E* p;
    int64_t ld, lim, K;
    bool vec;
    __device__ __forceinline__ void operator()(int o, int64_t k, double (&r)[4]) const {
        const E* q = p + k * ld + o;
        if (vec && k < K && o + 3 < lim) {
#pragma unroll
            for (int e = 0; e < 4; e += 16 / (int)sizeof(E)) {
                typedef E V __attribute__((ext_vector_type(16 / sizeof(E))));
                const V v = *reinterpret_cast<const V*>(q + e);
#pragma unroll
                for (int u = 0; u < 16 / (int)sizeof(E); ++u) r[e + u] = (double)v[u];
            }
            return;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (k < K && o + e < lim) ? (double)q[e] : 0.0;
    }
};

}  // namespace realq
