// Inverse of a lower-triangular tile (the "TRSM(L_ii^T, I)" of Phase 1, i.e.
// TRTRI).  A workgroup of 256 threads works on a tile, or on 64 columns of the
// corner, held in global memory (it stays in L2 while the workgroup runs); the
// products of 16 x 16 sub-blocks run on the FP64 matrix cores.
#pragma once
#include "common.hpp"

#define TO_LDD 17   // LDS leading dimension of 16-wide panels

// Lower-triangle tile index t -> (I, J), J <= I.
__device__ inline void tri_decode(int t, int& I, int& J) {
    int i = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (i * (i + 1) / 2 > t) --i;
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    I = i;
    J = t - i * (i + 1) / 2;
}

__device__ inline void neumaier(double& s, double& c, double x) {
    double t = s + x;
    if (fabs(s) >= fabs(x)) c += (s - t) + x;
    else c += (x - t) + s;
    s = t;
}

// LDS of the kernels around trtri_tile (per-wavefront 16 x 16 scratch) and
// trtri_columns (the inverses of up to 32 diagonal blocks).
#define TRTRI_SMEM_DOUBLES (32 * 16 * TO_LDD)

// X = L^{-1} for the m x m lower-triangular L (column-major, leading dimension
// ldl), m a multiple of 16, m <= 512.  X is written whole (upper part 0).
// Diagonal 16 x 16 blocks are inverted by forward substitution, then the block
// diagonals d = 1, 2, ... follow from X_IJ = -X_II sum_{K=J}^{I-1} L_IK X_KJ,
// every block of one diagonal in parallel.  Returns 1 in *bad (all threads) if
// a diagonal entry of L is not positive or is NaN.
__device__ __forceinline__ void trtri_tile(const double* L, int64_t ldl, double* X, int64_t ldx, int m,
                                  double* smem, int* bad) {
    __shared__ int s_bad;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wv = t >> 6;
    const int nblk = m / 16;
    if (t == 0) s_bad = 0;
    __syncthreads();
    // zero the blocks above the block diagonal
    for (int idx = t; idx < m * m; idx += 256) {
        const int i = idx % m, j = idx / m;
        if ((j >> 4) > (i >> 4)) X[i + (int64_t)j * ldx] = 0.0;
    }
    // 1. diagonal blocks, one column per lane
    for (int base = 0; base < nblk; base += 4) {
        const int blk = base + wv;
        if (blk < nblk && lane < 16) {
            const int o = 16 * blk;
            const int j = lane;
            double x[16];
            bool badl = false;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                double s = (i == j) ? 1.0 : 0.0;
#pragma unroll
                for (int k = 0; k < i; ++k) s -= L[(o + i) + (int64_t)(o + k) * ldl] * x[k];
                const double lii = L[(o + i) + (int64_t)(o + i) * ldl];
                if (!(lii > 0.0)) badl = true;
                x[i] = (i >= j) ? s / lii : 0.0;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) X[(o + i) + (int64_t)(o + j) * ldx] = x[i];
            if (badl) s_bad = 1;
        }
    }
    __syncthreads();
    // 2. block diagonals
    double* sT = smem + wv * 16 * TO_LDD;
    const int li = lane & 15, lk = lane >> 4;
    for (int dlt = 1; dlt < nblk; ++dlt) {
        const int ntask = nblk - dlt;
        for (int base = 0; base < ntask; base += 4) {
            const int J = base + wv;
            const bool act = J < ntask;
            const int I = J + dlt;
            dbl4 acc = {0.0, 0.0, 0.0, 0.0};
            if (act) {
                for (int K = J; K < I; ++K) {
#pragma unroll
                    for (int kk = 0; kk < 16; kk += 4) {
                        const double av = L[(16 * I + li) + (int64_t)(16 * K + kk + lk) * ldl];
                        const double bv = X[(16 * K + kk + lk) + (int64_t)(16 * J + li) * ldx];
                        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) sT[li * TO_LDD + 4 * r + lk] = acc[r];
            }
            __syncthreads();
            if (act) {
                dbl4 out = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int kk = 0; kk < 16; kk += 4) {
                    const double av = -X[(16 * I + li) + (int64_t)(16 * I + kk + lk) * ldx];
                    const double bv = sT[li * TO_LDD + kk + lk];
                    out = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, out, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    X[(16 * I + 4 * r + lk) + (int64_t)(16 * J + li) * ldx] = out[r];
            }
            __syncthreads();
        }
    }
    *bad = s_bad;
}


// Columns 64 s .. 64 s + 63 of X = L^{-1} for the m x m lower-triangular L, m a
// multiple of 16, m <= 512, by one workgroup: the inverses of the 16 x 16
// diagonal blocks from the first of these columns on go to LDS (16 lanes
// each), then wavefront v follows block column J = 4 s + v down, X_IJ = -X_II
// sum_{K=J}^{I-1} L_IK X_KJ.  A product on the matrix cores comes out as the
// operand of the next.  The block columns are independent: a corner of order
// 413 took one workgroup 600 us, its seven together take 70.
__device__ __forceinline__ void trtri_columns(const double* L, int64_t ldl, double* X, int64_t ldx, int m, int s,
                                              double* smem, int* bad) {
    __shared__ int s_bad;
    const int t = threadIdx.x;
    const int lane = t & 63, wv = t >> 6, li = lane & 15, lk = lane >> 4;
    const int nblk = m / 16, j0 = 4 * s;
    if (t == 0) s_bad = 0;
    __syncthreads();
    for (int idx = t; idx < 64 * s * 64; idx += 256) {   // rows above the column block
        const int j = 64 * s + idx / (64 * s);
        if (j < m) X[idx % (64 * s) + (int64_t)j * ldx] = 0.0;
    }
    for (int blk = j0 + 4 * wv + lk; blk < nblk; blk += 16) {
        const int o = 16 * blk, j = li;
        double x[16];
        bool badl = false;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            double v = (i == j) ? 1.0 : 0.0;
#pragma unroll
            for (int k = 0; k < i; ++k) v -= L[(o + i) + (int64_t)(o + k) * ldl] * x[k];
            const double lii = L[(o + i) + (int64_t)(o + i) * ldl];
            if (!(lii > 0.0)) badl = true;
            x[i] = (i >= j) ? v / lii : 0.0;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) smem[(blk * 16 + i) * TO_LDD + j] = x[i];
        if (badl) s_bad = 1;
    }
    __syncthreads();
    const int J = j0 + wv;
    if (J < nblk) {
        double* C = X + (int64_t)(16 * J) * ldx;
        auto put = [&](int I, const dbl4& x) {
#pragma unroll
            for (int r = 0; r < 4; ++r) C[(16 * I + 4 * r + lk) + (int64_t)li * ldx] = x[r];
        };
        for (int I = j0; I < J; ++I) put(I, dbl4{0.0, 0.0, 0.0, 0.0});
        dbl4 x;   // the block above: element r is (4 r + lk, li), the next product's operand
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = smem[(J * 16 + 4 * r + lk) * TO_LDD + li];
        put(J, x);
        for (int I = J + 1; I < nblk; ++I) {
            const double* R = L + 16 * I + li;
            dbl4 acc = {0.0, 0.0, 0.0, 0.0};
            for (int K = J; K < I - 1; ++K)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(R[(int64_t)(16 * K + 4 * kk + lk) * ldl],
                                                              C[(16 * K + 4 * kk + lk) + (int64_t)li * ldx], acc, 0, 0, 0);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(R[(int64_t)(16 * (I - 1) + 4 * kk + lk) * ldl], x[kk], acc, 0, 0, 0);
            x = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                x = __builtin_amdgcn_mfma_f64_16x16x4f64(-smem[(I * 16 + li) * TO_LDD + 4 * kk + lk], acc[kk], x, 0, 0, 0);
            put(I, x);
        }
    }
    *bad = s_bad;
}
