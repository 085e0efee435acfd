// Cholesky factor and inverse of one 16 x 16 block by one wavefront, the block
// and both results in registers in the matrix cores' output layout (lane
// (lk, li) = (lane / 16, lane % 16) holds row 4 r + lk, column li in element
// r), so the block comes straight from the products that formed it and its
// rank-4 updates run on the matrix cores.
//
// Four pivots at a time.  Element q of the layout holds rows 4q .. 4q + 3, one
// per 16-lane row of the wavefront; those four rows are copied into every
// 16-lane row (f16_rows), and the four pivots are eliminated among them with
// each lane keeping its column: a multiplier is one DPP broadcast along the
// lane row and a product, with no LDS and no exchange between lane rows.  The
// rest of the block then takes one v_mfma_f64_16x16x4_f64, whose two operands
// are the eliminated rows as they stand (by symmetry).  The inverse W of the
// unit lower factor goes through the same row operations.
//
// The chain per pivot is a broadcast, a reciprocal (hardware estimate and two
// Newton steps), a product and an FMA.
#pragma once
#include "common.hpp"

// Value of lane K of this lane's 16-lane row (DPP row_newbcast:K).
template <int K>
__device__ __forceinline__ double f16_bcast(double v) {
    return __builtin_amdgcn_mov_dpp(v, 0x150 + K, 0xF, 0xF, true);
}

// g[k] = the value lane (k, li) holds, in every lane (.., li).
__device__ __forceinline__ void f16_rows(double v, double (&g)[4]) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
    const u2 a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);   // rows 0 1 0 1 | 2 3 2 3
    const u2 b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    const u2 a01 = __builtin_amdgcn_permlane16_swap(a.x, a.x, false, false);
    const u2 b01 = __builtin_amdgcn_permlane16_swap(b.x, b.x, false, false);
    const u2 a23 = __builtin_amdgcn_permlane16_swap(a.y, a.y, false, false);
    const u2 b23 = __builtin_amdgcn_permlane16_swap(b.y, b.y, false, false);
    g[0] = __builtin_bit_cast(double, ((uint64_t)b01.x << 32) | a01.x);
    g[1] = __builtin_bit_cast(double, ((uint64_t)b01.y << 32) | a01.y);
    g[2] = __builtin_bit_cast(double, ((uint64_t)b23.x << 32) | a23.x);
    g[3] = __builtin_bit_cast(double, ((uint64_t)b23.y << 32) | a23.y);
}

// sqrt(x) and 1/sqrt(x) from the hardware reciprocal square root and two
// Goldschmidt steps (a few ulp; the pivot decides nothing else).
__device__ __forceinline__ void f16_sqrt_rsqrt(double x, double& s, double& r) {
    const double r0 = __builtin_amdgcn_rsq(x);
    double g = x * r0, h = 0.5 * r0;
    double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    s = g;
    r = 2.0 * h;
}

__device__ __forceinline__ double f16_own(const double (&g)[4], int lk) {
    const double a = lk & 1 ? g[1] : g[0], b = lk & 1 ? g[3] : g[2];
    return lk & 2 ? b : a;
}

// Pivot 4 Q + K among the rows g (of the block) and w (of W).
template <int Q, int K>
__device__ __forceinline__ void f16_pivot(double (&g)[4], double (&w)[4], double (&d)[4], double (&rr)[4], int& fail) {
    d[K] = f16_bcast<4 * Q + K>(g[K]);
    double r = __builtin_amdgcn_rcp(d[K]);
    double e = fma(-d[K], r, 1.0);
    r = fma(r, e, r);
    e = fma(-d[K], r, 1.0);
    r = fma(r, e, r);
    rr[K] = r;
    if (!(d[K] > 0.0) && fail < 0) fail = 4 * Q + K;
    if constexpr (K < 1) {
        const double f = f16_bcast<4 * Q + 1>(g[K]) * r;
        g[1] = fma(-f, g[K], g[1]);
        w[1] = fma(-f, w[K], w[1]);
    }
    if constexpr (K < 2) {
        const double f = f16_bcast<4 * Q + 2>(g[K]) * r;
        g[2] = fma(-f, g[K], g[2]);
        w[2] = fma(-f, w[K], w[2]);
    }
    if constexpr (K < 3) {
        const double f = f16_bcast<4 * Q + 3>(g[K]) * r;
        g[3] = fma(-f, g[K], g[3]);
        w[3] = fma(-f, w[K], w[3]);
    }
}

// Rows 4 Q .. 4 Q + 3: t = U^T rows times their pivots, h = W's rows, dv the
// pivots (each this lane's row 4 Q + lk), and the rank-4 update of the rest.
template <int Q>
__device__ __forceinline__ void f16_group(dbl4& S, dbl4& W, double (&t)[4], double (&h)[4], double (&dv)[4], int& fail,
                                          int lk) {
    double g[4], w[4], d[4], rr[4];
    f16_rows(S[Q], g);
    f16_rows(W[Q], w);
    f16_pivot<Q, 0>(g, w, d, rr, fail);
    f16_pivot<Q, 1>(g, w, d, rr, fail);
    f16_pivot<Q, 2>(g, w, d, rr, fail);
    f16_pivot<Q, 3>(g, w, d, rr, fail);
    t[Q] = f16_own(g, lk);
    dv[Q] = f16_own(d, lk);
    h[Q] = f16_own(w, lk);
    if constexpr (Q < 3) {
        const double a = -(t[Q] * f16_own(rr, lk));
        S = __builtin_amdgcn_mfma_f64_16x16x4f64(a, t[Q], S, 0, 0, 0);
        W = __builtin_amdgcn_mfma_f64_16x16x4f64(a, h[Q], W, 0, 0, 0);
    }
}

// S: the block, both triangles.  l[q] = L(li, 4 q + lk) (zero above the
// diagonal), y[q] = Y(4 q + lk, li) with Y = L^{-1}.  fail (-1 on entry) gets
// the first column whose pivot is not positive.
__device__ __forceinline__ void f16_factor(dbl4 S, double (&l)[4], double (&y)[4], int& fail) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    dbl4 W;
#pragma unroll
    for (int r = 0; r < 4; ++r) W[r] = li == 4 * r + lk ? 1.0 : 0.0;
    double t[4], h[4], dv[4];
    f16_group<0>(S, W, t, h, dv, fail, lk);
    f16_group<1>(S, W, t, h, dv, fail, lk);
    f16_group<2>(S, W, t, h, dv, fail, lk);
    f16_group<3>(S, W, t, h, dv, fail, lk);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        double s, r;
        f16_sqrt_rsqrt(dv[q], s, r);
        const int k = 4 * q + lk;
        l[q] = li > k ? t[q] * r : (li == k ? s : 0.0);
        y[q] = h[q] * r;
    }
}
