// Cholesky factor and inverse of one 16 x 16 block by one wavefront, four
// columns (a group) at a time, the block in registers in the matrix cores'
// output layout (lane (lk, li) = (lane / 16, lane % 16) holds row 4 r + lk,
// column li in element r), so it comes straight from the products that formed
// it.
//
// For group q the 4 x 4 block of rows and columns 4q .. 4q + 3 is read into
// scalar registers and factored by every lane alike, L4; lane (k, 4 b + i)
// keeps the entry (i, k) of Y4 = L4^{-1}, which is the operand of
// v_mfma_f64_4x4x4_4b that makes the four rows of L^T out of the block's four
// rows as they lie, and those rows are both operands of the
// v_mfma_f64_16x16x4 that updates the rest.  The identity W goes through the
// same row operations and comes out as Y = L^{-1}; its products run in the
// shadow of the next group's scalar work.
//
// What bounds it is the number of instructions (about 90 per group, four
// cycles or more each) and the chain of 16 pivots: a reciprocal square root
// (hardware estimate and one step of third order), a product and an FMA each.
// Measured alone, one wavefront, L and Y: 3,010 cycles; one column per lane with
// DPP broadcasts, no matrix cores, took 4,450 for L.
#pragma once
#include "common.hpp"

// The value lane L holds, in a scalar register pair.
__device__ __forceinline__ double f16_lane(double v, int L) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, L), hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), L);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// 1 / sqrt(x): hardware estimate r (relative error below 2^-20) and one step
// of third order, r (1 + e / 2 + 3 e^2 / 8) with e = 1 - x r^2.
__device__ __forceinline__ double f16_rsqrt(double x) {
    const double r = __builtin_amdgcn_rsq(x);
    const double e = fma(-x, r * r, 1.0);
    return fma(r * e, fma(0.375, e, 0.5), r);
}

// Group Q of the block S (both triangles of the part not yet factored): t =
// L(li, 4 Q + lk) (meaningless above the diagonal), y4 as above, S updated.
// fail: the first of the block's columns whose pivot is not
// positive, if none was found before (-1).
// pt, py4, py: those of the group before, whose products into W run here, behind
// the reads of S (in front of them they would hold up the wavefront).
template <int Q>
__device__ __forceinline__ void f16_group(dbl4& S, dbl4& W, double& t, double& y4, double pt, double py4, double& py,
                                          int& fail) {
    // the lane opaque: what depends on it is formed here, not kept in
    // registers (or scratch memory) across the caller's loop
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int li = lane & 15, lk = lane >> 4;
    const double a00 = f16_lane(S[Q], 4 * Q), a10 = f16_lane(S[Q], 4 * Q + 1);
    const double a20 = f16_lane(S[Q], 4 * Q + 2), a30 = f16_lane(S[Q], 4 * Q + 3);
    double a11 = f16_lane(S[Q], 16 + 4 * Q + 1), a21 = f16_lane(S[Q], 16 + 4 * Q + 2);
    double a31 = f16_lane(S[Q], 16 + 4 * Q + 3), a22 = f16_lane(S[Q], 32 + 4 * Q + 2);
    double a32 = f16_lane(S[Q], 32 + 4 * Q + 3), a33 = f16_lane(S[Q], 48 + 4 * Q + 3);
    if constexpr (Q > 0) {
        __builtin_amdgcn_sched_barrier(0);
        py = __builtin_amdgcn_mfma_f64_4x4x4f64(py4, W[Q - 1], 0.0, 0, 0, 0);
        W = __builtin_amdgcn_mfma_f64_16x16x4f64(-pt, py, W, 0, 0, 0);
    }
    // column lk of Y4 in this lane: L4 y = e_lk
    const double r0 = f16_rsqrt(a00);
    const double l10 = a10 * r0, l20 = a20 * r0, l30 = a30 * r0;
    a11 = fma(-l10, l10, a11);
    const double r1 = f16_rsqrt(a11);
    a21 = fma(-l20, l10, a21);
    a31 = fma(-l30, l10, a31);
    a22 = fma(-l20, l20, a22);
    a32 = fma(-l30, l20, a32);
    a33 = fma(-l30, l30, a33);
    const double l21 = a21 * r1, l31 = a31 * r1;
    a22 = fma(-l21, l21, a22);
    const double r2 = f16_rsqrt(a22);
    a32 = fma(-l31, l21, a32);
    a33 = fma(-l31, l31, a33);
    const double l32 = a32 * r2;
    a33 = fma(-l32, l32, a33);
    const double r3 = f16_rsqrt(a33);
    double y0 = lk == 0 ? r0 : 0.0;
    double y1 = fma(-l10, y0, lk == 1 ? 1.0 : 0.0) * r1;
    double y2 = fma(-l21, y1, fma(-l20, y0, lk == 2 ? 1.0 : 0.0)) * r2;
    double y3 = fma(-l32, y2, fma(-l31, y1, fma(-l30, y0, lk == 3 ? 1.0 : 0.0))) * r3;
    asm volatile("" : "+v"(y0), "+v"(y1), "+v"(y2), "+v"(y3));   // selected, not branched around
    y4 = li & 2 ? (li & 1 ? y3 : y2) : (li & 1 ? y1 : y0);
    t = __builtin_amdgcn_mfma_f64_4x4x4f64(y4, S[Q], 0.0, 0, 0, 0);
    if constexpr (Q < 3) S = __builtin_amdgcn_mfma_f64_16x16x4f64(-t, t, S, 0, 0, 0);
    // the pivots are the same in every lane
    int k = -1;
    if (__ballot(!(a33 > 0.0))) k = 4 * Q + 3;
    if (__ballot(!(a22 > 0.0))) k = 4 * Q + 2;
    if (__ballot(!(a11 > 0.0))) k = 4 * Q + 1;
    if (__ballot(!(a00 > 0.0))) k = 4 * Q;
    fail = fail < 0 ? k : fail;
}

// S: the block, both triangles.  l[q] = L(li, 4 q + lk) (meaningless above the
// diagonal), y[q] = Y(4 q + lk, li) with Y = L^{-1}.  The first column whose
// pivot is not positive, or -1.
__device__ __forceinline__ int f16_factor(dbl4 S, double (&l)[4], double (&y)[4]) {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    dbl4 W;
#pragma unroll
    for (int r = 0; r < 4; ++r) W[r] = (lane & 15) == 4 * r + (lane >> 4) ? 1.0 : 0.0;
    int fail = -1;
    double g[4], none = 0.0;
    f16_group<0>(S, W, l[0], g[0], 0.0, 0.0, none, fail);
    f16_group<1>(S, W, l[1], g[1], l[0], g[0], y[0], fail);
    f16_group<2>(S, W, l[2], g[2], l[1], g[1], y[1], fail);
    f16_group<3>(S, W, l[3], g[3], l[2], g[2], y[2], fail);
    y[3] = __builtin_amdgcn_mfma_f64_4x4x4f64(g[3], W[3], 0.0, 0, 0, 0);
    return fail;
}
