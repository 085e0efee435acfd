// HIP kernels and the C ABI (include/stiles.h) of the band-plus-arrowhead
// selected inversion: tile Cholesky with log det, then Phase 1 and Phase 2 of
// the two-phase backward recurrence (arXiv 2504.19171, Sec. III-D).
//
// Execution: every step is enqueued on the caller's stream; each kernel below
// covers one tile-level operation over all the tiles it can do at once.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <atomic>
#include <mutex>
#include <vector>

#include "../../include/stiles.h"
#include "common.hpp"
#include "gemm_block.hpp"
#include "tile_ops.hpp"
#include "persist.hpp"
#include "wave_gemm.hpp"
#include "factor.hpp"
#include "phase2.hpp"

#define NT 256
#define WS_HEAD 256  // bytes reserved at the start of every workspace (info and scheduler words)

// ---------------------------------------------------------------------------
// Layout
// ---------------------------------------------------------------------------
static int make_layout(int64_t n, int64_t bandwidth, int64_t arrow, int32_t tile, stiles_layout* o) {
    if (n < 1) return -1;
    if (bandwidth < 0) return -2;
    if (arrow < 0 || arrow >= n || arrow > 512) return -3;
    if (!(tile == 64 || tile == 128 || tile == 192 || tile == 256)) return -4;
    memset(o, 0, sizeof(*o));
    o->n = n; o->bandwidth = bandwidth; o->arrow = arrow; o->tile = tile;
    o->nb = n - arrow;
    o->w = std::min<int64_t>(bandwidth, o->nb - 1);
    o->nt = (o->nb + tile - 1) / tile;
    int64_t bt = (o->w + tile - 1) / tile;
    if (bt > o->nt - 1) bt = o->nt - 1;
    o->bt = (int32_t)bt;
    o->arrow_ld = (int32_t)((arrow + 15) / 16 * 16);
    const int64_t b2 = (int64_t)tile * tile;
    o->off_band = 0;
    o->off_arrow = o->nt * (o->bt + 1) * b2;
    o->off_corner = o->off_arrow + o->nt * (int64_t)o->arrow_ld * tile;
    o->total_doubles = o->off_corner + (int64_t)o->arrow_ld * o->arrow_ld;
    return 0;
}

static Lay to_dev(const stiles_layout& s) {
    Lay l;
    l.nb = s.nb; l.w = s.w; l.nt = s.nt;
    l.off_band = s.off_band; l.off_arrow = s.off_arrow; l.off_corner = s.off_corner;
    l.total = s.total_doubles;
    l.b = s.tile; l.bt = s.bt; l.ap = s.arrow_ld; l.a = (int)s.arrow;
    return l;
}

static int grid_for(int64_t work) {
    int64_t g = (work + NT - 1) / NT;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

// ---------------------------------------------------------------------------
// Small kernels
// ---------------------------------------------------------------------------
__global__ void k_zero_ints(int* p, int64_t n) {
    for (int64_t i = threadIdx.x + (int64_t)blockIdx.x * blockDim.x; i < n; i += (int64_t)blockDim.x * gridDim.x) p[i] = 0;
}
// Pack the canonical band form into the tile layout (every double written).
// Workgroup g < N (B+1) writes band tile g = J (B+1) + d, i.e. tile (J+d, J);
// the next N write the arrow tiles J; the rest the corner's 64 x 64 blocks.
//
// A band tile is written 32 columns at a time through LDS.  Column c of tile
// (J+d, J) holds A[(J+d) b + r, J b + c]; in the band form that is
// ab[d b + r - c, J b + c] (on and below the diagonal) and ab[c - r, J b + r]
// (above it, diagonal tiles only).  For a fixed band-form row k both are 32
// consecutive doubles over the 32 columns, so the reads run along the rows of
// ab, the block is assembled in LDS and written out column by column: both
// sides coalesced.  The arrow tiles go the same way: a row of P is contiguous,
// a tile column is contiguous.
#define PACK_CB 32
#define PACK_RB 256
#define PACK_SMEM_DOUBLES (PACK_CB * (PACK_RB + 1))
#define PACK_U 8   // loads in flight per thread
__global__ __launch_bounds__(NT) void k_pack(const double* __restrict__ ab, const double* __restrict__ P,
                                            const double* __restrict__ C, double* __restrict__ T, Lay L) {
    __shared__ double blk[PACK_SMEM_DOUBLES];   // [c][r]: column c at c * b (band) or c * (rows + 1) (arrow)
    const int b = L.b;
    const int64_t nband = L.nt * (int64_t)(L.bt + 1);
    const int64_t g = blockIdx.x;
    const int tid = threadIdx.x;
    if (g < nband) {
        const int64_t J = g / (L.bt + 1);
        const int d = (int)(g % (L.bt + 1));
        double* O = T + g * (int64_t)b * b;
        const bool live = J + d < L.nt;
        const int64_t i0 = (J + d) * b, j0 = J * b;   // global row / column of the tile's (0, 0)
        if (b == 64) {
            // 64 x 64 tiles: the staging costs more than it saves (each block
            // would read 95 band-form rows for 64 tile rows); thread t writes
            // row t % 64 of columns t / 64, t / 64 + 4, ...
            // (every load from a valid address, the unused ones dropped: a
            // load under a branch would wait before the next one issues)
            const int r = tid % 64;
            const int64_t i = i0 + r;
            constexpr int NQ = 64 / (NT / 64);
            double v[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int64_t j = j0 + tid / 64 + q * (NT / 64);
                const int64_t k = i >= j ? i - j : j - i, lo = i >= j ? j : i;
                const bool ok = live && i < L.nb && j < L.nb && k <= L.w;
                v[q] = ab[ok ? k * L.nb + lo : 0];
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int c = tid / 64 + q * (NT / 64);
                const int64_t j = j0 + c;
                const bool in = live && i < L.nb && j < L.nb;
                const int64_t k = i >= j ? i - j : j - i;
                O[r + c * 64] = (in && k <= L.w) ? v[q] : ((live && !in && i == j) ? 1.0 : 0.0);
            }
            return;
        }
        for (int cb = 0; cb < b; cb += PACK_CB) {
            // defaults: 0, or 1 on the diagonal past the band part (identity padding)
            for (int e = tid; e < PACK_CB * b; e += NT) {
                const int c = e / b, r = e % b;
                blk[e] = (live && d == 0 && r == cb + c && i0 + r >= L.nb) ? 1.0 : 0.0;
            }
            __syncthreads();
            if (live) {
                // on and below the diagonal: k = d b + r - c', c' = cb + c.
                // PACK_U loads per thread are issued before their LDS stores,
                // each from a valid address (the unused ones dropped): a load
                // under a branch would wait before the next one issues.
                const int klo = imax_(0, d * b - cb - (PACK_CB - 1)), khi = imin_((int)L.w, d * b + b - 1 - cb);
                const int n = (khi - klo + 1) * PACK_CB;
                for (int e0 = tid; e0 < n; e0 += NT * PACK_U) {
                    double v[PACK_U];
                    int at[PACK_U];
#pragma unroll
                    for (int q = 0; q < PACK_U; ++q) {
                        const int e = e0 + q * NT;
                        const int k = klo + e / PACK_CB, c = e % PACK_CB;
                        const int r = k - d * b + cb + c;
                        const int64_t j = j0 + cb + c;
                        const bool ok = e < n && r >= 0 && r < b && i0 + r < L.nb && j < L.nb;
                        v[q] = ab[ok ? (int64_t)k * L.nb + j : 0];
                        at[q] = ok ? c * b + r : -1;
                    }
#pragma unroll
                    for (int q = 0; q < PACK_U; ++q)
                        if (at[q] >= 0) blk[at[q]] = v[q];
                }
                if (d == 0) {
                    // above the diagonal: k = c' - r >= 1, value ab[k, j0 + r]
                    const int khi2 = imin_((int)L.w, cb + PACK_CB - 1);
                    const int n2 = imax_(khi2, 0) * PACK_CB;
                    for (int e0 = tid; e0 < n2; e0 += NT * PACK_U) {
                        double v[PACK_U];
                        int at[PACK_U];
#pragma unroll
                        for (int q = 0; q < PACK_U; ++q) {
                            const int e = e0 + q * NT;
                            const int k = 1 + e / PACK_CB, c = e % PACK_CB;
                            const int r = cb + c - k;
                            const bool ok = e < n2 && r >= 0 && j0 + cb + c < L.nb;
                            v[q] = ab[ok ? (int64_t)k * L.nb + j0 + r : 0];
                            at[q] = ok ? c * b + r : -1;
                        }
#pragma unroll
                        for (int q = 0; q < PACK_U; ++q)
                            if (at[q] >= 0) blk[at[q]] = v[q];
                    }
                }
            }
            __syncthreads();
            for (int e = tid; e < PACK_CB * b; e += NT) O[(int64_t)cb * b + e] = blk[e];
            __syncthreads();
        }
    } else if (g < nband + L.nt) {
        const int64_t J = g - nband;
        double* O = T + L.arrow(J);
        const int ap = L.ap;
        const int64_t j0 = J * b;
        for (int cb = 0; cb < b; cb += PACK_CB) {
            for (int rb = 0; rb < ap; rb += PACK_RB) {
                const int nr = imin_(PACK_RB, ap - rb);
                // rows r of P over the block's 32 columns (contiguous), into [c][r]
                for (int e0 = tid; e0 < nr * PACK_CB; e0 += NT * PACK_U) {
                    double v[PACK_U];
                    int at[PACK_U];
                    bool ok[PACK_U];
#pragma unroll
                    for (int q = 0; q < PACK_U; ++q) {
                        const int e = e0 + q * NT;
                        const int r = e / PACK_CB, c = e % PACK_CB;
                        const int64_t j = j0 + cb + c;
                        ok[q] = rb + r < L.a && j < L.nb;
                        v[q] = P[ok[q] ? (int64_t)(rb + r) * L.nb + j : 0];
                        at[q] = e < nr * PACK_CB ? c * (nr + 1) + r : -1;
                    }
#pragma unroll
                    for (int q = 0; q < PACK_U; ++q)
                        if (at[q] >= 0) blk[at[q]] = ok[q] ? v[q] : 0.0;
                }
                __syncthreads();
                for (int e = tid; e < nr * PACK_CB; e += NT) {
                    const int c = e / nr, r = e % nr;
                    O[(int64_t)(cb + c) * ap + rb + r] = blk[c * (nr + 1) + r];
                }
                __syncthreads();
            }
        }
    } else {
        // the corner in 64 x 64 blocks through LDS (C by rows, the tile by
        // columns); by one workgroup it took a corner of 413 rows 300 us
        double* O = T + L.corner();
        const int ap = L.ap, nab = arrow_blocks(ap), q = (int)(g - nband - L.nt);
        const int r0 = 64 * (q % nab), c0 = 64 * (q / nab);
        for (int e = tid; e < 64 * 64; e += NT) {
            const int r = e >> 6, c = e & 63;
            blk[r * 65 + c] = r0 + r < L.a && c0 + c < L.a ? C[(int64_t)(r0 + r) * L.a + c0 + c]
                                                           : (r0 + r == c0 + c ? 1.0 : 0.0);
        }
        __syncthreads();
        for (int e = tid; e < 64 * 64; e += NT) {
            const int r = e & 63, c = e >> 6;
            if (r0 + r < ap && c0 + c < ap) O[r0 + r + (int64_t)(c0 + c) * ap] = blk[r * 65 + c];
        }
    }
}

// Zero the band tiles (J+d, J) with J+d >= N (outside the matrix); block bid
// of nblk.
__device__ inline void zero_unused_body(double* T, const Lay& L, int bid, int nblk) {
    const int64_t b2 = (int64_t)L.b * L.b;
    const int64_t ntail = (int64_t)L.bt * (L.bt + 1) / 2;  // tiles J+d >= N
    const int64_t tot = ntail * b2;
    for (int64_t idx = bid * (int64_t)NT + threadIdx.x; idx < tot; idx += (int64_t)nblk * NT) {
        const int64_t t = idx / b2, e = idx % b2;
        // enumerate (J, d) with J = N-1-m, d = m+1..B, m = 0..B-1
        int64_t m = 0, cnt = t;
        while (cnt >= L.bt - m) { cnt -= L.bt - m; ++m; }
        const int64_t J = L.nt - 1 - m, d = m + 1 + cnt;
        T[L.band(J, (int)d) + e] = 0.0;
    }
}

// ---------------------------------------------------------------------------
// Factor kernels
// ---------------------------------------------------------------------------

// Compensated sum over a wavefront of the pairs (s, c) of its lanes, joined
// pairwise in a fixed order (the lower lane of each pair is the left operand,
// so all lanes agree).
__device__ inline void neumaier_join(double& s, double& c) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double qs = __shfl_xor(s, o), qc = __shfl_xor(c, o);
        const bool lo = (lane & o) == 0;
        const double a = lo ? s : qs, b = lo ? qs : s;
        const double t = a + b;
        const double e = (fabs(a) >= fabs(b)) ? (a - t) + b : (b - t) + a;
        c = (lo ? c + qc : qc + c) + e;
        s = t;
    }
}

// After the band: the strict upper triangles of its diagonal tiles set to 0
// (the layout's convention for L; nothing in the factorization reads them),
// eight workgroups per tile, b/8 columns each; the first of the eight also
// sums the tile's part of log det, 2 log L_jj over its columns (off the
// chain, which only stores the diagonal).
__device__ inline void factor_tail_body(double* Lm, const Lay& L, int bid, double* ldp) {
    const int64_t J = bid >> 3;
    const int cw = L.b / 8, c0 = (bid & 7) * cw;
    double* T = (double*)(GLOBAL_AS double*)(Lm + L.band(J, 0));
    for (int c = c0; c < c0 + cw; ++c)
        for (int i = threadIdx.x; i < c; i += NT) T[i + (int64_t)c * L.b] = 0.0;
    if ((bid & 7) == 0 && threadIdx.x < 64) {
        double s = 0.0, c = 0.0;
        for (int j = threadIdx.x; j < L.b; j += 64) neumaier(s, c, 2.0 * log(T[j * (int64_t)(L.b + 1)]));
        neumaier_join(s, c);
        if (threadIdx.x == 0) {
            ldp[2 * J] = s;
            ldp[2 * J + 1] = c;
        }
    }
}

// The corner is factored by the same persistent kernel, as a dense matrix of 64
// x 64 tiles in the workspace (its own layout: a_p rows rounded up to 64, the
// rest the identity).  a_p <= 512, so the copies there and back are 2 MB at
// most.  (One workgroup on the corner in place took 49 / 220 / 640 us at a_p =
// 64 / 208 / 416.)
__host__ __device__ inline Lay corner_lay(const Lay& L) {
    Lay c;
    const int nab = arrow_blocks(L.ap);
    c.nb = 64 * nab;
    c.w = nab > 0 ? c.nb - 1 : 0;
    c.nt = nab;
    c.b = 64;
    c.bt = nab > 0 ? nab - 1 : 0;
    c.ap = c.a = 0;
    c.off_band = 0;
    c.off_arrow = c.off_corner = c.total = (int64_t)nab * nab * 64 * 64;
    return c;
}
// Workgroups that copy the corner there (its lower 64 x 64 blocks) and back
// (all blocks, and one for the log det).
__host__ __device__ inline int corner_in_blocks(const Lay& L) {
    const int nab = arrow_blocks(L.ap);
    return nab * (nab + 1) / 2;
}
__host__ __device__ inline int corner_out_blocks(const Lay& L) {
    const int nab = arrow_blocks(L.ap);
    return nab > 0 ? nab * nab + 1 : 0;
}
__device__ inline void corner_in_body(const double* Lm, const Lay& L, int bid, double* T) {
    const Lay K = corner_lay(L);
    int r, c;
    tri_decode(bid, r, c);
    const double* A = (const double*)(GLOBAL_AS const double*)(Lm + L.corner());
    double* O = (double*)(GLOBAL_AS double*)(T + K.band(c, r - c));
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
        const int i = 64 * r + (e & 63), j = 64 * c + (e >> 6);
        O[e] = i < L.ap && j < L.ap ? A[i + (int64_t)j * L.ap] : (i == j ? 1.0 : 0.0);
    }
}
__device__ inline void corner_out_body(double* Lm, const Lay& L, int bid, const double* T, double* ldp) {
    const Lay K = corner_lay(L);
    const int nab = arrow_blocks(L.ap);
    T = (const double*)(GLOBAL_AS const double*)T;
    if (bid == nab * nab) {
        if (threadIdx.x >= 64) return;
        double s = 0.0, c = 0.0;
        for (int j = threadIdx.x; j < 64 * nab; j += 64) neumaier(s, c, 2.0 * log(T[K.band(j >> 6, 0) + (j & 63) * 65]));
        neumaier_join(s, c);
        if (threadIdx.x == 0) {
            ldp[2 * L.nt] = s;
            ldp[2 * L.nt + 1] = c;
        }
        return;
    }
    const int r = bid % nab, c = bid / nab;
    double* A = (double*)(GLOBAL_AS double*)(Lm + L.corner());
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
        const int i = 64 * r + (e & 63), j = 64 * c + (e >> 6);
        if (i < L.ap && j < L.ap) A[i + (int64_t)j * L.ap] = i >= j ? T[K.band(c, r - c) + e] : 0.0;
    }
}
// Workgroups 8 N .. of the tail: the corner's copy.
__host__ __device__ inline int factor_tail_blocks(const Lay& L) { return (int)(8 * L.nt) + corner_in_blocks(L); }
__device__ inline void factor_tail(double* Lm, const Lay& L, int bid, double* ldp, double* T) {
    if (bid < 8 * L.nt) factor_tail_body(Lm, L, bid, ldp);
    else corner_in_body(Lm, L, (int)(bid - 8 * L.nt), T);
}
__global__ __launch_bounds__(NT) void k_factor_tail(double* Lm, Lay L, double* ldp, double* T) {
    factor_tail(Lm, L, blockIdx.x, ldp, T);
}

// Group and index inside it of task t of one matrix.
__device__ inline void fac_ticket(const FacCtx& x, int t, int& c, int& u) {
    const int f4 = fac_full4(x);
    if (f4 > 0) {
        const int n = fac_group(x, 0), n4 = 3 * n + fac_group(x, 3);
        const int q = t / n4;
        if (q < f4 / 4) {
            const int r = t - q * n4, e = imin_(r / n, 3);
            c = 4 * q + e;
            u = r - e * n;
            return;
        }
        t -= f4 / 4 * n4;
    }
    for (c = f4; c < x.nc - 1; ++c) {
        const int n = fac_group(x, c);
        if (t < n) break;
        t -= n;
    }
    u = t;
}

// The band factor of one matrix in one persistent launch (factor.hpp): the first
// tickets are the chains, the next ones the tasks.
// Until no tickets are left (true) or the kernel must stop.
template <int LD>
__device__ inline bool fac_run(const FacCtx& x, int ntask, const Sched& sc, FacSmem& sm, int* info) {
    if (threadIdx.x == 0) sm.dead = 0;
    const int nch = fac_chains(x);
    for (;;) {
        const int g = sched_next(sc, nch + ntask, &sm.sh);
        if (g < 0) return true;
        if (g < nch) {
            if (!fac_chain(x, sc, sm, g, nch > 1 ? g + 1 : x.nc, info, g == sc.withhold)) return false;
            continue;
        }
        int c, u;
        fac_ticket(x, g - nch, c, u);
        if (!fac_task<LD>(x, sc, sm, c, u, g)) return false;
    }
}
template <int LD>
__global__ __launch_bounds__(FAC_NT, 2) void k_factor_all(FacCtx x, int ntask, Sched sc, int* info) {
    __shared__ FacSmem sm;
    fac_run<LD>(x, ntask, sc, sm, info);
}

// Final log det (compensated sum of the partial pairs in a fixed order: each
// lane of the one wavefront every 64th, then joined) and info.
__device__ inline void factor_final_body(const double* ldp, int nparts, const int* info_ws, const int* err,
                                         double* logdet, int* info) {
    double s = 0.0, c = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 64) {
        neumaier(s, c, ldp[2 * i]);
        neumaier(s, c, ldp[2 * i + 1]);
    }
    neumaier_join(s, c);
    if (threadIdx.x != 0) return;
    const int f = (*err != 0) ? *err : *info_ws;
    *info = (f == 0x7fffffff) ? 0 : f;
    *logdet = (f == 0x7fffffff) ? (s + c) : __builtin_nan("");
}
// The corner back to its place; the workgroup that has its log det then ends the
// factor.
__global__ __launch_bounds__(NT) void k_corner_out(double* Lm, Lay L, const double* T, double* ldp, const int* info_ws,
                                                   const int* err, double* logdet, int* info) {
    corner_out_body(Lm, L, blockIdx.x, T, ldp);
    if ((int)blockIdx.x != corner_out_blocks(L) - 1 || threadIdx.x >= 64) return;
    __threadfence();   // the corner's own part of ldp, by lane 0
    factor_final_body(ldp, (int)L.nt + 1, info_ws, err, logdet, info);
}
__global__ __launch_bounds__(64) void k_factor_final(const double* ldp, int nparts, const int* info_ws, const int* err,
                                                     double* logdet, int* info) {
    factor_final_body(ldp, nparts, info_ws, err, logdet, info);
}

// ---------------------------------------------------------------------------
// Selected-inversion kernels
// ---------------------------------------------------------------------------

// Phase 1, diagonal tiles: X_J = L_JJ^{-1} ("TRSM(L_ii^T, I)"), stored in the
// diagonal slots of the workspace; the corner inverse likewise, one workgroup
// per 64 columns.  A tile takes one workgroup per 64 columns too when the whole
// matrix (a range of its columns counts as the whole) has at most 512 of them,
// two per CU, or when a tile has 64 (79 tiles of 256: 131 against 188 us; 27,000
// of 64: 0.87 against 1.13 ms), else one, which inverts each diagonal block once
// (391 of 256: 303 against 442 us).
__host__ __device__ inline int trtri_per(const Lay& L) { return L.b == 64 || L.nt * (L.b / 64) <= 512 ? L.b / 64 : 1; }
__host__ __device__ inline int trtri_blocks(const Lay& L) { return (int)L.nt * trtri_per(L) + arrow_blocks(L.ap); }
__device__ inline void trtri_body(const double* Lm, double* W, const Lay& L, int* info, int bid, double* smem) {
    const int per = trtri_per(L);
    const int64_t J = bid / per;
    int bad;
    if (J < L.nt && L.b > 64 && per == 1) {
        trtri_tile(Lm + L.band(J, 0), L.b, W + L.band(J, 0), L.b, L.b, smem, &bad);
    } else {
        const bool band = J < L.nt;
        const int64_t at = band ? L.band(J, 0) : L.corner();
        const int m = band ? L.b : L.ap, s = band ? bid % per : (int)(bid - L.nt * per);
        trtri_columns(Lm + at, m, W + at, m, m, s, smem, &bad);
    }
    if (threadIdx.x == 0 && bad) atomicExch(info, STILES_EBADL);
}
// (j0: first tile column; the launches of a selection start there)
__global__ __launch_bounds__(NT, 2) void k_trtri_all(const double* Lm, double* W, Lay L, int* info, int64_t j0) {
    __shared__ double smem[TRTRI_SMEM_DOUBLES];
    trtri_body(Lm, W, L, info, (int)(blockIdx.x + j0 * trtri_per(L)), smem);
}

// Rows of the panel below tile J (band tiles J+1..J+s, then the arrow tile),
// 64-row block blk.
__device__ inline void panel_rows(const Lay& L, double* base, int64_t J, int blk, double*& C,
                                  int64_t& ld, int& valid) {
    const int nb64 = L.b / 64;
    const int s = L.s(J);
    if (blk < s * nb64) {
        const int d = 1 + blk / nb64, rb = blk % nb64;
        C = base + L.band(J, d) + rb * 64;
        ld = L.b;
        valid = 64;
    } else {
        const int rb = blk - s * nb64;
        C = base + L.arrow(J) + rb * 64;
        ld = L.ap;
        valid = imin_(64, L.ap - rb * 64);
    }
}

// Phase 1, off-diagonal tiles: Lhat_{k,J} = L_{k,J} X_J for the band tiles
// k = J+1..J+s and the arrow tile ("TRMM").  Grid: (J, 64-row block, col block).
__device__ inline void trmm_body(const double* Lm, double* W, const Lay& L, int bid, double* smem) {
    const int nb64 = L.b / 64;
    const int nab = arrow_blocks(L.ap);
    const int rows_max = L.bt * nb64 + nab;
    const int64_t J = bid / (rows_max * nb64);
    const int r = (int)(bid % (rows_max * nb64));
    const int blk = r / nb64, cb = r % nb64;
    const int s = L.s(J);
    if (blk >= s * nb64 + nab) return;
    double* Cw;
    int64_t ld;
    int valid;
    panel_rows(L, W, J, blk, Cw, ld, valid);
    const double* Cl = Lm + (Cw - W);
    const double* X = W + L.band(J, 0);
    const int k0 = cb * 64;
    GAcc g;
    gacc_zero(g);
    gemm_acc(g, opnd(Cl + (int64_t)k0 * ld, ld, 0, valid), opnd(X + k0 + (int64_t)k0 * L.b, L.b, 0, 64),
             L.b - k0, smem);
    gemm_store(g, smem, 1.0, 0.0, nullptr, 0, Cw + (int64_t)k0 * ld, ld, valid, 64);
}
__global__ __launch_bounds__(NT) void k_trmm_all(const double* Lm, double* W, Lay L, int64_t j0) {
    __shared__ double smem[GB_SMEM_DOUBLES];
    const int nb64 = L.b / 64;
    trmm_body(Lm, W, L, xcd_block((int)blockIdx.x, (int)gridDim.x) + (int)(j0 * (L.bt * nb64 + arrow_blocks(L.ap)) * nb64),
              smem);
}

// Phase 2 initial value of each diagonal tile, "LAUUM": Sigma_JJ = X_J^T X_J
// (and the corner Sigma_AA = X_A^T X_A, which is final).  Lower 64 x 64
// blocks, mirrored so the tiles are full symmetric.  Blocks are numbered
// densely: lauum_per(L) per band tile column, then the corner's
// (lauum_corner(L), none without an arrow).
__host__ __device__ inline int lauum_per(const Lay& L) {
    const int nb64 = L.b / 64;
    return nb64 * (nb64 + 1) / 2;
}
__host__ __device__ inline int lauum_corner(const Lay& L) {
    const int nab = arrow_blocks(L.ap);
    return L.ap > 0 ? nab * (nab + 1) / 2 : 0;
}
// blocks of tile columns j0.. and the corner
__host__ __device__ inline int64_t lauum_blocks(const Lay& L, int64_t j0) {
    return (L.nt - j0) * (int64_t)lauum_per(L) + lauum_corner(L);
}
// (W in layout K, Sigma in layout L: the same tiles, no more of them in K)
__device__ inline void lauum_body(const double* W, const Lay& K, double* S, const Lay& L, int64_t bid, double* smem) {
    const int per = lauum_per(L);
    const int64_t nband = L.nt * (int64_t)per;
    const double* X;
    double* O;
    int m;
    int64_t ld;
    int t;
    if (bid < nband) {
        const int64_t J = bid / per;
        t = (int)(bid % per);
        X = W + K.band(J, 0); O = S + L.band(J, 0); m = L.b; ld = L.b;
    } else {
        t = (int)(bid - nband);
        if (t >= lauum_corner(L)) return;
        X = W + K.corner(); O = S + L.corner(); m = L.ap; ld = L.ap;
    }
    int rb, cb;
    tri_decode(t, rb, cb);
    const int k0 = rb * 64;
    const int va = imin_(64, m - rb * 64), vb = imin_(64, m - cb * 64);
    GAcc g;
    gacc_zero(g);
    gemm_acc(g, opnd(X + k0 + (int64_t)rb * 64 * ld, ld, 1, va), opnd(X + k0 + (int64_t)cb * 64 * ld, ld, 0, vb),
             m - k0, smem);
    gemm_store_sym(g, smem, 1.0, 0.0, nullptr, 0, O + rb * 64 + (int64_t)cb * 64 * ld,
                   O + cb * 64 + (int64_t)rb * 64 * ld, ld, rb == cb, va, vb);
}
__global__ __launch_bounds__(NT) void k_lauum_all(const double* W, double* S, Lay L, int64_t j0) {
    __shared__ double smem[GB_SMEM_DOUBLES];
    lauum_body(W, L, S, L, xcd_block((int)blockIdx.x, (int)gridDim.x) + j0 * lauum_per(L), smem);
}

// Before a selected inverse (Sigma in layout L): no task done, first ticket, no
// error, and zero the band tiles of S that lie outside the matrix (S null: none).
__device__ inline void selinv_setup_body(const Lay& L, double* S, int* cnt, int* ticket, int* err, int* info, int bid, int nblk) {
    p2_setup_body(L, cnt, ticket, err, info, bid, nblk);
    if (S && L.bt > 0) zero_unused_body(S, L, bid, nblk);
}
__global__ __launch_bounds__(NT) void k_selinv_setup(Lay L, double* S, int* cnt, int* ticket, int* err, int* info) {
    selinv_setup_body(L, S, cnt, ticket, err, info, blockIdx.x, gridDim.x);
}
static int selinv_setup_grid(const Lay& L) {
    return std::min(grid_for((int64_t)L.bt * (L.bt + 1) / 2 * L.b * L.b), 2048);
}
__global__ __launch_bounds__(P2Cfg<8>::NTH, 2) void k_phase2(P2 p, Sched sc) {
    __shared__ __attribute__((aligned(128))) double smem[P2Cfg<8>::SMEM];
    __shared__ int sh[2];
    p2_run<8>(p, sc, smem, sh);
}

__global__ void k_selinv_final(const int* info_ws, const int* err, int* info) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *info = (*err != 0) ? *err : *info_ws;
}

// ---------------------------------------------------------------------------
// Batched form: many independent matrices per launch
// ---------------------------------------------------------------------------
// Every launch of the single-matrix path becomes one launch over all the
// matrices of a batch that have work in it: a table of segments maps each
// workgroup to (matrix, workgroup index within that matrix's share), and
// every matrix keeps its own tickets, counters and workspace, so the tasks,
// their decomposition and their arithmetic are those of the single-matrix
// path, matrix by matrix (results are identical bit for bit).

// Sub-buffers of a factor workspace (shared by both forms).
struct FactorWs {
    int* winfo;     // first failing column (atomicMin), 0x7fffffff when none
    int* err;       // scheduler error word
    int* ticket;
    double* ldp;    // log det partial pairs, N + 2 of them
    int* cticket;   // the corner's
    double* Tc;     // the corner's tiles (corner_lay)
    double* Ycd;    // its 16 x 16 diagonal-block inverses
    double* Yd;     // 16 x 16 diagonal-block inverses of every L_JJ
    int* flags;     // fac_ints(L) flags, then the corner's
};
__host__ __device__ inline FactorWs factor_ws(const Lay& L, char* ws) {
    FactorWs f;
    f.winfo = (int*)ws;
    f.err = f.winfo + 16;
    f.ticket = f.winfo + 32;
    f.cticket = f.winfo + 48;
    f.ldp = (double*)(ws + WS_HEAD);
    f.Tc = f.ldp + 2 * (L.nt + 2);
    const int64_t nab = arrow_blocks(L.ap);
    f.Ycd = f.Tc + nab * nab * 64 * 64;
    f.Yd = f.Ycd + nab * 64 * 16;
    f.flags = (int*)(f.Yd + L.nt * (int64_t)L.b * 16);
    return f;
}

// Before a factor: no failing column, no error, first ticket, no flag up.
__device__ inline void factor_setup_body(const Lay& L, const FactorWs& f, int64_t at, int64_t step) {
    if (at == 0) {
        *f.winfo = 0x7fffffff;
        *f.err = 0;
        *f.ticket = 0;
        *f.cticket = 0;
    }
    const int64_t n = fac_ints(L) + fac_ints(corner_lay(L));
    for (int64_t i = at; i < n; i += step) f.flags[i] = 0;
}
// The corner's factor.
__host__ __device__ inline FacCtx corner_ctx(const Lay& L, const FactorWs& f) {
    FacCtx x = fac_ctx(corner_lay(L), f.Tc, f.Ycd, f.flags ? f.flags + fac_ints(L) : nullptr);
    x.col0 = (int)L.nb;
    return x;
}
__global__ __launch_bounds__(NT) void k_factor_setup(Lay L, FactorWs f) {
    factor_setup_body(L, f, threadIdx.x + (int64_t)blockIdx.x * NT, (int64_t)NT * gridDim.x);
}

// Sub-buffers of a selinv workspace.
struct SelinvWs {
    int* winfo;     // selinv info
    int* ticket;    // Phase 2 ticket counter
    int* err;       // Phase 2 scheduler error word
    double* W;      // Phase 1 tiles (tile layout)
    int* flags;     // Phase 2 ready counters
};
__host__ __device__ inline SelinvWs selinv_ws(const Lay& L, char* ws) {
    SelinvWs v;
    v.winfo = (int*)ws;
    v.ticket = v.winfo + 16;
    v.err = v.winfo + 32;
    v.W = (double*)(ws + WS_HEAD);
    v.flags = (int*)(v.W + L.total);
    return v;
}

// Phase 2 on tile columns J >= jf of Sigma in layout L, W in layout K (the same
// tiles, no more of them).
__host__ __device__ inline P2 make_p2(double* S, const Lay& L, const double* W, const Lay& K, int* cnt, int ntasks, int64_t jf) {
    P2 p;
    p.S = S;
    p.W = W;
    p.L = L;
    p.btw = K.bt;
    p.warrow = K.off_arrow;
    p.cnt = cnt;
    p.ntasks = ntasks;
    const int64_t N = L.nt;
    p.klast = imin_(L.b, (int)((L.b + K.w - K.bt * (int64_t)L.b + 31) / 32 * 32));
    p.jf = (int)jf;
    const int64_t qr = L.bt > 1 ? L.bt : 1, ql = imax64(N - 1 - jf, 0);
    p.q0 = (int)(ql < qr ? ql : qr);
    p.off_q0 = (int)p2_base(L, p.q0);
    p.g_tasks = p2_group_tasks(L, N - 1 - p.q0, jf);
    return p;
}

// One matrix of a batch, as the device sees it.
struct BInst {
    Lay L;
    const double* A;
    double* Lm;
    double* S;
    double* logdet;
    int* info;        // [0] factor, [1] selinv
    char* ws;         // this matrix's workspace (factor or selinv layout)
    int fac_ntask;    // factor task count
    int fac_nticket;  // ... and with the chains
    int p2_tasks;     // Phase 2 task count
    int nparts;       // log det partial pairs (factor_nparts)
};
// Workgroups [first, next first) of a launch belong to matrix inst; a table
// of nseg segments ends with a sentinel holding the launch's grid size.
struct BSeg {
    int inst;
    int first;
};
struct BArgs {
    const BInst* bi;
    const BSeg* seg;
    int nseg;
    int64_t spin_limit;
};
__device__ inline int bseg_find(const BSeg* seg, int nseg, int b) {
    int lo = 0, hi = nseg;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (seg[mid].first <= b) lo = mid; else hi = mid;
    }
    return lo;
}
// the matrix of logical block B, B's index within the matrix's share, and
// the share's size
#define BATCH_DECODE_AT(a, I, bid, nblk, B)                                    \
    const int b_ = (B);                                                        \
    const int q_ = bseg_find((a).seg, (a).nseg, b_);                           \
    const BInst& I = (a).bi[(a).seg[q_].inst];                                 \
    const int bid = b_ - (a).seg[q_].first;                                    \
    const int nblk = (a).seg[q_ + 1].first - (a).seg[q_].first;                \
    (void)nblk
// ... of this workgroup.  (The XCD grouping of the single-matrix Phase 1
// products, applied to the batched ones, made them slower: kb_lauum 597 ->
// 762 us per pass; not used here.)
#define BATCH_DECODE(a, I, bid, nblk) BATCH_DECODE_AT(a, I, bid, nblk, (int)blockIdx.x)

// Factor set-up of every matrix (eight workgroups each).
__global__ __launch_bounds__(NT) void kb_factor_setup(const BInst* bi) {
    const BInst& I = bi[blockIdx.x >> 3];
    factor_setup_body(I.L, factor_ws(I.L, I.ws), threadIdx.x + (int64_t)(blockIdx.x & 7) * NT, 8 * NT);
}

// The band factors of matrices [k0, k1), at most KB_SLICE a launch: each starts
// on its own share of the workgroups (two or more), with its own tickets, the
// first of which is its chain.  (With one queue over all matrices, chunk after
// chunk, in 97 launches, 64 matrices took 22.3 ms; this takes 14.3.)  A
// workgroup whose matrix has no tickets left
// joins the one with the most work left (tasks, times the length of their sums)
// among those whose chain is under way: so no workgroup becomes a chain that
// waits for others that have all become chains too.
#define KB_SLICE 128
template <int LD>
__global__ __launch_bounds__(FAC_NT, 2) void kb_factor(BArgs a, int k0, int k1, int* err) {
    __shared__ FacSmem sm;
    sched_batch(
        a.seg[bseg_find(a.seg, a.nseg, (int)blockIdx.x)].inst, k0, k1, err, &sm.sh,
        [&](int k) {
            const BInst& I = a.bi[k];
            const FactorWs f = factor_ws(I.L, I.ws);
            Sched sc;
            sc.ticket = f.ticket;
            sc.err = err;
            sc.spin_limit = a.spin_limit;
            sc.withhold = -1;
            const FacCtx x = fac_ctx(I.L, I.Lm, f.Yd, f.flags);
            return fac_run<LD>(x, I.fac_ntask, sc, sm, f.winfo);
        },
        [&](int m) {
            const BInst& M = a.bi[m];
            const int t = ld_coh_i(factor_ws(M.L, M.ws).ticket), left = M.fac_nticket - t;
            return t > 0 && left > 0 ? (float)left * (float)(fac_wc(M.L) + 4) : 0.0f;
        });
}

__global__ __launch_bounds__(NT) void kb_factor_tail(BArgs a) {
    BATCH_DECODE(a, I, bid, nblk);
    const FactorWs f = factor_ws(I.L, I.ws);
    factor_tail(I.Lm, I.L, bid, f.ldp, f.Tc);
}

// The corners, each on its own workgroups with its own tickets.  (A matrix's
// workgroups follow one another in the launch, so whichever of them are
// resident, those of the first unfinished one are.)
__global__ __launch_bounds__(FAC_NT, 2) void kb_corner(BArgs a, int* err) {
    __shared__ FacSmem sm;
    BATCH_DECODE(a, I, bid, nblk);
    const FactorWs f = factor_ws(I.L, I.ws);
    Sched sc;
    sc.ticket = f.cticket;
    sc.err = err;
    sc.spin_limit = a.spin_limit;
    sc.withhold = -1;
    const FacCtx x = corner_ctx(I.L, f);
    fac_run<FAC_WIDE>(x, (int)fac_tasks(x), sc, sm, f.winfo);
}
__global__ __launch_bounds__(NT) void kb_corner_out(BArgs a) {
    BATCH_DECODE(a, I, bid, nblk);
    const FactorWs f = factor_ws(I.L, I.ws);
    corner_out_body(I.Lm, I.L, bid, f.Tc, f.ldp);
}

__global__ __launch_bounds__(64) void kb_factor_final(const BInst* bi, const int* err) {
    const BInst& I = bi[blockIdx.x];
    const FactorWs f = factor_ws(I.L, I.ws);
    factor_final_body(f.ldp, I.nparts, f.winfo, err, I.logdet, I.info);
}

// Selinv set-up of every matrix.
__global__ __launch_bounds__(NT) void kb_selinv_setup(BArgs a) {
    BATCH_DECODE(a, I, bid, nblk);
    const SelinvWs v = selinv_ws(I.L, I.ws);
    selinv_setup_body(I.L, I.S, v.flags, v.ticket, v.err, v.winfo, bid, nblk);
}

__global__ __launch_bounds__(NT, 2) void kb_trtri(BArgs a) {
    __shared__ double smem[TRTRI_SMEM_DOUBLES];
    BATCH_DECODE(a, I, bid, nblk);
    const SelinvWs v = selinv_ws(I.L, I.ws);
    trtri_body(I.Lm, v.W, I.L, v.winfo, bid, smem);
}

__global__ __launch_bounds__(NT) void kb_trmm(BArgs a) {
    __shared__ double smem[GB_SMEM_DOUBLES];
    BATCH_DECODE(a, I, bid, nblk);
    trmm_body(I.Lm, selinv_ws(I.L, I.ws).W, I.L, bid, smem);
}

__global__ __launch_bounds__(NT) void kb_lauum(BArgs a) {
    __shared__ double smem[GB_SMEM_DOUBLES];
    BATCH_DECODE(a, I, bid, nblk);
    lauum_body(selinv_ws(I.L, I.ws).W, I.L, I.S, I.L, bid, smem);
}

// What `tasks` Phase 2 tasks of a matrix weigh: the length of their sums and a
// fixed cost of 256 (shares by task counts: 64 matrices 17.6 against 16.8 ms, 8
// served ones 8.5 against 7.7; without the fixed cost 17.5 and 7.5, but 1.55
// against 1.43 for 32 narrow ones).
__host__ __device__ inline double p2_work(const Lay& L, int tasks) { return (double)tasks * (double)(L.bt * L.b + L.ap + 256); }
#define P2_WIDE_TASKS 512.0
// Phase 2 of every matrix in one persistent launch: each matrix starts on its
// own share of the workgroups, with its own tickets, and a workgroup whose
// matrix has no tickets left joins the one with the most work left (tasks, times
// the length of their sums).
template <int NW>
__global__ __launch_bounds__(P2Cfg<NW>::NTH, 2) void kb_phase2(BArgs a, int count) {
    __shared__ __attribute__((aligned(128))) double smem[P2Cfg<NW>::SMEM];
    __shared__ int sh[2];
    sched_batch(
        a.seg[bseg_find(a.seg, a.nseg, (int)blockIdx.x)].inst, 0, count, nullptr, &sh[1],
        [&](int k) {
            const BInst& I = a.bi[k];
            const SelinvWs v = selinv_ws(I.L, I.ws);
            Sched sc;
            sc.ticket = v.ticket;
            sc.err = v.err;
            sc.spin_limit = a.spin_limit;
            sc.withhold = -1;
            return p2_run<NW>(make_p2(I.S, I.L, v.W, I.L, v.flags, I.p2_tasks, 0), sc, smem, sh);
        },
        [&](int m) {
            const BInst& M = a.bi[m];
            const SelinvWs u = selinv_ws(M.L, M.ws);
            const int left = ld_coh_i(u.err) == 0 ? M.p2_tasks - ld_coh_i(u.ticket) : 0;
            return left > 0 ? (float)p2_work(M.L, left) : 0.0f;
        });
}

__global__ void kb_selinv_final(const BInst* bi) {
    if (threadIdx.x != 0) return;
    const BInst& I = bi[blockIdx.x];
    const SelinvWs v = selinv_ws(I.L, I.ws);
    *(I.info + 1) = (*v.err != 0) ? *v.err : *v.winfo;
}

// ---------------------------------------------------------------------------
// Trace of a product over the tile pattern (gradient of log det)
// ---------------------------------------------------------------------------
// sum_ij S_ij B_ij over the real entries of two symmetric matrices stored on
// the same tile pattern: a diagonal band tile and the corner hold both
// triangles (weight 1 each), a band tile below the diagonal and an arrow tile
// the strictly lower part (weight 2: the upper part mirrors it); padding
// (rows or columns past nb in the band, past a in the arrow) is left out.
// The buffer is one tile column after another (of b or a_p doubles), so each of
// the TP_BLOCKS workgroups' wavefronts takes every TP_WAVES-th of them, in a
// fixed order, and works out its place once (element by element the divisions
// bounded the pass: 1.07 ms where reading both buffers, 1.9 GB each, takes
// 0.72); k_trace_final adds the parts (compensated, in a fixed order), so the
// result does not depend on timing.
#define TP_BLOCKS 1024
#define TP_WAVES (TP_BLOCKS * (NT / 64))
__global__ __launch_bounds__(NT) void k_trace_part(const double* __restrict__ S, const double* __restrict__ B, Lay L,
                                                   double* part) {
    __shared__ double red[NT];
    const int lane = threadIdx.x & 63;
    const int64_t per = (int64_t)(L.bt + 1) * L.b;   // columns of a tile column's band tiles
    const int64_t nband = L.nt * per, narrow = L.ap > 0 ? L.nt * (int64_t)L.b : 0, n = nband + narrow + L.ap;
    double acc = 0.0;
    for (int64_t u = blockIdx.x * (NT / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); u < n; u += TP_WAVES) {
        int64_t at, rows;   // where the column starts, its rows that count
        double wgt = 2.0;
        if (u < nband) {
            const int64_t J = u / per;
            const int v = (int)(u - J * per), d = v / L.b, c = v - d * L.b;
            at = u * L.b;
            rows = J * L.b + c < L.nb ? L.nb - (J + d) * L.b : 0;
            rows = rows < 0 ? 0 : rows > L.b ? L.b : rows;
            if (d == 0) wgt = 1.0;
        } else if (u < nband + narrow) {
            at = L.off_arrow + (u - nband) * L.ap;
            rows = u - nband < L.nb ? L.a : 0;
        } else {
            at = L.off_corner + (u - nband - narrow) * L.ap;
            rows = u - nband - narrow < L.a ? L.a : 0;
            wgt = 1.0;
        }
        for (int64_t r = lane; r < rows; r += 256) {
            double x[4], y[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {   // (each load from the column, those past its end dropped)
                const int64_t i = at + (r + 64 * q < rows ? r + 64 * q : r);
                x[q] = S[i];
                y[q] = B[i];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (r + 64 * q < rows) acc = fma(wgt * x[q], y[q], acc);
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int o = NT / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}
__global__ __launch_bounds__(64) void k_trace_final(const double* part, double* out) {
    double s = 0.0, c = 0.0;
    for (int g = threadIdx.x; g < TP_BLOCKS; g += 64) neumaier(s, c, part[g]);
    neumaier_join(s, c);
    if (threadIdx.x == 0) *out = s + c;
}

// ---------------------------------------------------------------------------
// Selected entries read off the tile layout
// ---------------------------------------------------------------------------
// out[k] = Sigma(ij[2k], ij[2k+1]) (either order: Sigma is symmetric); NaN
// for a pair outside the tile pattern of L or outside the matrix.
__global__ __launch_bounds__(NT) void k_gather(const double* S, Lay L, const int64_t* ij, int64_t count, double* out) {
    const int64_t n = L.nb + L.a;
    for (int64_t k = blockIdx.x * (int64_t)NT + threadIdx.x; k < count; k += (int64_t)gridDim.x * NT) {
        int64_t i = ij[2 * k], j = ij[2 * k + 1];
        if (i < j) { const int64_t t = i; i = j; j = t; }
        double v = __builtin_nan("");
        if (j >= 0 && i < n) {
            if (j < L.nb) {
                const int64_t J = j / L.b, c = j - J * L.b;
                if (i < L.nb) {
                    const int64_t I = i / L.b;
                    if (I - J <= L.bt) v = S[L.band(J, (int)(I - J)) + (i - I * L.b) + c * L.b];
                } else {
                    v = S[L.arrow(J) + (i - L.nb) + c * L.ap];
                }
            } else {
                v = S[L.corner() + (i - L.nb) + (j - L.nb) * L.ap];
            }
        }
        out[k] = v;
    }
}

// ---------------------------------------------------------------------------
// Full inversion (every entry of A^{-1})
// ---------------------------------------------------------------------------
// The recurrence of Phase 2 over every tile row instead of the rows of S(J):
//   Sigma_{i,J} = -sum_{k in S(J)} Sigma_{i,k} Lhat_{k,J}   for all i below J,
// (Sec. III-D; the full-inversion case of Sec. III-B).  So it is Phase 2 with
// Sigma in the layout of a dense band (every tile below the diagonal) and W in
// L's own; the sums run over W's tiles only.  (A launch per column and for its
// diagonal tile took 46 us a column at w 256, a 37, tile 128; this takes 15.)
__host__ __device__ inline Lay full_lay(const Lay& L) {
    Lay F = L;
    F.bt = (int)(L.nt - 1);
    F.w = L.nb - 1;
    F.off_band = 0;
    F.off_arrow = L.nt * L.nt * (int64_t)L.b * L.b;
    F.off_corner = F.off_arrow + L.nt * (int64_t)L.ap * L.b;
    F.total = F.off_corner + (int64_t)L.ap * L.ap;
    return F;
}
__global__ __launch_bounds__(NT) void k_inv_lauum(const double* W, Lay L, double* S, Lay F) {
    __shared__ double smem[GB_SMEM_DOUBLES];
    lauum_body(W, L, S, F, xcd_block((int)blockIdx.x, (int)gridDim.x), smem);
}

// The n x n output from Sigma's tiles (layout F), a pair of mirrored 64 x 64
// blocks per workgroup, the upper one through LDS.  Block rows and columns of
// the band lie in one tile each; a block may end in arrow rows.
__global__ __launch_bounds__(NT) void k_inv_compact(const double* __restrict__ S, Lay F, double* __restrict__ O) {
    __shared__ double blk[64 * 65];
    const int64_t n = F.nb + F.a;
    int rb, cb;
    tri_decode((int)blockIdx.x, rb, cb);
    const int64_t i0 = 64 * (int64_t)rb, j0 = 64 * (int64_t)cb;
    const int64_t It = i0 / F.b, Jt = j0 / F.b;
    const bool low = i0 < F.nb && j0 < F.nb;   // some of the block is of the band
    const double* T = S + (low ? F.band(Jt, (int)(It - Jt)) + (i0 - It * F.b) + (j0 - Jt * F.b) * F.b : 0);
    const double* R = S + (j0 < F.nb ? F.arrow(Jt) + (j0 - Jt * F.b) * F.ap : 0);
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
        const int r = e & 63, c = e >> 6;
        int64_t i = i0 + r, j = j0 + c;
        if (i >= n || j >= n) continue;
        double v;
        if (i < F.nb && j < F.nb) v = T[r + c * F.b];
        else if (j < F.nb) v = R[(i - F.nb) + c * (int64_t)F.ap];
        else if (i >= F.nb) v = S[F.corner() + (i - F.nb) + (j - F.nb) * F.ap];
        else v = S[F.arrow(Jt) + (j - F.nb) + (i - Jt * F.b) * F.ap];   // above the diagonal of a diagonal block
        O[i + j * n] = v;
        blk[r * 65 + c] = v;
    }
    if (rb == cb) return;
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
        const int c = e & 63, r = e >> 6;
        const int64_t i = i0 + r, j = j0 + c;
        if (i < n && j < n) O[j + i * n] = blk[r * 65 + c];
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

// Pure matrix-core throughput: every wavefront runs 8 independent chains of
// v_mfma_f64_16x16x4_f64 (2048 flops each), so the matrix pipe of its SIMD
// never waits on a result.  sink keeps the compiler from dropping the work.
#define PEAK_CHAINS 8
__global__ __launch_bounds__(NT) void k_mfma_peak(double* sink, int iters) {
    const int lane = threadIdx.x & 63;
    const double a = 1.0 + 1e-3 * lane, b = 1.0 - 1e-3 * lane;
    dbl4 acc[PEAK_CHAINS];
#pragma unroll
    for (int c = 0; c < PEAK_CHAINS; ++c) acc[c] = dbl4{0.0, 0.0, 0.0, (double)c};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int c = 0; c < PEAK_CHAINS; ++c) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[c], 0, 0, 0);
    }
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < PEAK_CHAINS; ++c) s += acc[c][0] + acc[c][1] + acc[c][2] + acc[c][3];
    sink[blockIdx.x * (int64_t)NT + threadIdx.x] = s;
}

static inline hipStream_t S_(void* s) { return (hipStream_t)s; }

#define HIPCHK(x)                              \
    do {                                       \
        if ((x) != hipSuccess) return STILES_EHIP; \
    } while (0)
#define LAUNCHCHK()                                       \
    do {                                                  \
        if (hipGetLastError() != hipSuccess) return STILES_EHIP; \
    } while (0)


// Optional per-kernel event timing (see stiles_timing_enable in stiles.h).
struct EvRec {
    hipEvent_t a, b;
    int kind;
};
static std::mutex g_tmu;
static std::atomic<bool> g_timing{false};
static std::vector<EvRec> g_ev;

static hipEvent_t tm_begin(hipStream_t st) {
    if (!g_timing.load(std::memory_order_relaxed)) return nullptr;
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    if (hipEventRecord(e, st) != hipSuccess) {
        (void)hipEventDestroy(e);
        return nullptr;
    }
    return e;
}

static void tm_end(hipEvent_t a, int kind, hipStream_t st) {
    if (!a) return;
    hipEvent_t b;
    if (hipEventCreate(&b) != hipSuccess) {
        (void)hipEventDestroy(a);
        return;
    }
    (void)hipEventRecord(b, st);
    std::lock_guard<std::mutex> g(g_tmu);
    g_ev.push_back({a, b, kind});
}

static void tm_drop() {
    std::lock_guard<std::mutex> g(g_tmu);
    for (auto& e : g_ev) {
        (void)hipEventSynchronize(e.b);
        (void)hipEventDestroy(e.a);
        (void)hipEventDestroy(e.b);
    }
    g_ev.clear();
}

#define LAUNCH(kind, kern, grid, block, shm, st, ...)                           \
    do {                                                                       \
        hipEvent_t _tm = tm_begin(st);                                         \
        hipLaunchKernelGGL(kern, grid, block, shm, st, __VA_ARGS__);           \
        if (hipGetLastError() != hipSuccess) return STILES_EHIP;               \
        tm_end(_tm, kind, st);                                                 \
    } while (0)

// Per-device facts used to size persistent launches (queried once).
struct DevInfo {
    int cus = 0;
    int64_t clock_khz = 0;
};
static std::mutex g_dmu;
static DevInfo g_dev[64];

static int dev_info(DevInfo* out) {
    int d = 0;
    if (hipGetDevice(&d) != hipSuccess || d < 0 || d >= 64) return STILES_EHIP;
    std::lock_guard<std::mutex> g(g_dmu);
    if (g_dev[d].cus == 0) {
        int cus = 0, khz = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, d) != hipSuccess) return STILES_EHIP;
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, d) != hipSuccess) return STILES_EHIP;
        g_dev[d].cus = cus > 0 ? cus : 1;
        g_dev[d].clock_khz = khz > 0 ? khz : 100000;
    }
    *out = g_dev[d];
    return 0;
}

// Wait limit of the device-side spin loops: STILES_SPIN_LIMIT_MS (default
// 4000 ms).  STILES_DEBUG_WITHHOLD=<ticket> makes that task skip its ready
// signal, to exercise the timeout path.
static int64_t spin_limit_ticks(const DevInfo& di) {
    double ms = 4000.0;
    if (const char* e = getenv("STILES_SPIN_LIMIT_MS")) {
        const double v = atof(e);
        if (v > 0) ms = v;
    }
    return (int64_t)(ms * (double)di.clock_khz);
}

static int debug_withhold() {
    if (const char* e = getenv("STILES_DEBUG_WITHHOLD")) return atoi(e);
    return -1;
}

// Workgroups of one matrix's factor: the chain and the tasks of FAC_AHEAD
// chunks.  A workgroup that holds a ticket further ahead than its task can
// start only polls, and the polls share the memory channels of the flags that
// the chain itself waits for.  Measured with 24 and without a limit: 5.46 and
// 5.55 ms at nb 30,011, w 501, tile 192; the same at w 1,024 and above, where
// 24 chunks' tasks fill the chip anyway.  Below 16 some widths lose (w 2,001,
// nb 100,000: 21.1 ms with 24, 24.6 with 8).
#define FAC_AHEAD 24
// With a chain per chunk (wc 0) the chains wait for nothing: as many as fit.
static int fac_grid(const FacCtx& x, int most) {
    if (fac_chains(x) > 1) return most;
    int g = 0;
    for (int c = 0; c < std::min(4, x.nc); ++c) g = std::max(g, fac_group(x, c));
    return std::min(most, 2 + FAC_AHEAD * g);
}


// log det partial pairs: one per band tile column, one for the corner
static int factor_nparts(const Lay& L) { return (int)L.nt + (L.ap > 0 ? 1 : 0); }

// Workgroups of a corner's factor: the chain and up to 31 for its tasks (at
// most eight block rows).
static int corner_grid(const Lay& L) {
    if (L.ap == 0) return 0;
    const FacCtx x = fac_ctx(corner_lay(L), nullptr, nullptr, nullptr);
    return (int)std::min<int64_t>(fac_chains(x) + fac_tasks(x), 32);
}

static int64_t p2_total_tasks(const Lay& L) {
    int64_t t = 0;
    for (int64_t J = 0; J < L.nt; ++J) t += p2_group_tasks(L, J, 0);
    return t;
}

// Batch plan: layouts, the table area at the start of the workspace (the
// matrices, then the launch segment tables) and each matrix's workspace.
static size_t align256(size_t x) { return (x + 255) / 256 * 256; }
// The kernels read their workspaces with 16-byte loads, and a caller may place
// one anywhere: it is used from its first multiple of 16 bytes on, and every
// workspace size has that much to spare.
#define WS_ALIGN 16
static char* ws_base(void* p) { return (char*)(((uintptr_t)p + WS_ALIGN - 1) / WS_ALIGN * WS_ALIGN); }
struct BPlan {
    std::vector<stiles_layout> lay;
    std::vector<size_t> off;   // workspace offset of each matrix
    size_t table_f = 0;        // bytes of the factor's table area (at the start of the workspace)
    size_t table = 0;          // bytes of both table areas (the selected inverse's follows the factor's)
    size_t total = 0;
};
// factor workspace (FactorWs): head (info, error words) + log det partials
// (N + 2 pairs) + the corner's tiles and diagonal-block inverses + the 16 x 16
// diagonal-block inverses of every L_JJ + the flags of the persistent launches.
// Never less than one tile, which callers may count on.
static size_t fws_bytes(const stiles_layout& l) {
    const Lay L = to_dev(l);
    const size_t n = WS_HEAD + sizeof(double) * (size_t)(2 * (l.nt + 2)) +
                     sizeof(double) * (size_t)(corner_lay(L).total + arrow_blocks(L.ap) * 64 * 16 + l.nt * (int64_t)l.tile * 16) +
                     sizeof(int) * (size_t)(fac_ints(L) + fac_ints(corner_lay(L)));
    return std::max(n, sizeof(double) * (size_t)l.tile * (size_t)l.tile);
}
// selinv workspace (SelinvWs): head (info, ticket, error words), the Phase 1
// tiles (inverted diagonal tiles, Lhat, corner inverse) in the tile layout,
// then the Phase 2 counters.
static size_t sws_bytes(const stiles_layout& l) {
    return WS_HEAD + sizeof(double) * (size_t)l.total_doubles + sizeof(int) * (size_t)((l.bt + 2) * l.nt);
}
static size_t batch_nseg(int count) {
    return 6 * ((size_t)count + 1) + ((size_t)count + KB_SLICE - 1) / KB_SLICE;
}
static int batch_plan(const stiles_batch_item* items, int count, bool need_sigma, BPlan& pl) {
    pl.lay.resize(count);
    pl.off.resize(count);
    for (int k = 0; k < count; ++k) {
        const stiles_batch_item& it = items[k];
        if (make_layout(it.n, it.bandwidth, it.arrow, it.tile, &pl.lay[k])) return -1;
        if (it.reserved != 0 || !it.A || !it.L || !it.logdet || !it.info) return -1;
        if (need_sigma && (!it.Sigma || it.Sigma == it.L)) return -1;
        if (need_sigma && p2_total_tasks(to_dev(pl.lay[k])) > 0x7fffffff) return -1;
    }
    // segment tables of at most six per-matrix launches and a sentinel per
    // launch of the factor, then the factor's error word
    const size_t nseg = batch_nseg(count);
    pl.table_f = align256(sizeof(BInst) * (size_t)count) + align256(sizeof(BSeg) * nseg) + align256(sizeof(int));
    pl.table = pl.table_f + align256(sizeof(BInst) * (size_t)count) + align256(sizeof(BSeg) * nseg);
    size_t o = pl.table;
    for (int k = 0; k < count; ++k) {
        pl.off[k] = o;
        o += align256(std::max(fws_bytes(pl.lay[k]), sws_bytes(pl.lay[k])));
    }
    pl.total = WS_ALIGN + o;
    return 0;
}

// Segment table builder: workgroup shares of one launch.
struct SegTab {
    size_t begin = 0;
    int grid = 0;
    void start(size_t b) { begin = b; grid = 0; }
    void add(std::vector<BSeg>& all, int inst, int blocks) {
        if (blocks <= 0) return;
        all.push_back({inst, grid});
        grid += blocks;
    }
    int finish(std::vector<BSeg>& all) {   // returns the segment count
        const int n = (int)(all.size() - begin);
        all.push_back({-1, grid});
        return n;
    }
};

extern "C" {

#ifdef STILES_TASK_TRACE
int stiles_debug_trace_read(unsigned long long* host, size_t n_tasks) {
    if (n_tasks > STILES_TRACE_MAX) n_tasks = STILES_TRACE_MAX;
    return hipMemcpyFromSymbol(host, HIP_SYMBOL(g_trace), STILES_TRACE_SLOTS * n_tasks * sizeof(unsigned long long), 0,
                               hipMemcpyDeviceToHost) == hipSuccess ? 0 : STILES_EHIP;
}
#endif

int stiles_version(void) { return 100; }

int stiles_timing_enable(int on) {
    tm_drop();
    g_timing.store(on != 0);
    return 0;
}

int stiles_timing_collect(double* ms, int64_t* launches) {
    if (!ms) return -1;
    if (!launches) return -2;
    for (int k = 0; k < STILES_TK_COUNT; ++k) {
        ms[k] = 0.0;
        launches[k] = 0;
    }
    std::lock_guard<std::mutex> g(g_tmu);
    int rc = 0;
    for (auto& e : g_ev) {
        float t = 0.0f;
        if (hipEventSynchronize(e.b) != hipSuccess || hipEventElapsedTime(&t, e.a, e.b) != hipSuccess) rc = STILES_EHIP;
        if (e.kind >= 0 && e.kind < STILES_TK_COUNT) {
            ms[e.kind] += (double)t;
            launches[e.kind] += 1;
        }
        (void)hipEventDestroy(e.a);
        (void)hipEventDestroy(e.b);
    }
    g_ev.clear();
    return rc;
}


const char* stiles_strerror(int code) {
    if (code == 0) return "success";
    if (code > 0) return "matrix is not positive definite (info = failing column, 1-based)";
    switch (code) {
        case -1: return "invalid argument 1";
        case -2: return "invalid argument 2";
        case -3: return "invalid argument 3";
        case -4: return "invalid argument 4";
        case -5: return "invalid argument 5";
        case -6: return "invalid argument 6";
        case -7: return "invalid argument 7";
        case -8: return "invalid argument 8";
        case -9: return "invalid argument 9";
        case -10: return "invalid argument 10";
        case -11: return "invalid argument 11";
        case STILES_EHIP: return "HIP runtime error";
        case STILES_ETIMEOUT: return "device wait exceeded its spin limit";
        case STILES_EBADL: return "a diagonal entry of L is not positive";
        case STILES_ENOTBUILT: return "library not built or not loaded";
        default: return "invalid argument";
    }
}

int stiles_layout_init(int64_t n, int64_t bandwidth, int64_t arrow, int32_t tile, stiles_layout* out) {
    if (!out) return -5;
    return make_layout(n, bandwidth, arrow, tile, out);
}

size_t stiles_factor_workspace_bytes(const stiles_layout* lay) { return lay ? WS_ALIGN + fws_bytes(*lay) : 0; }

size_t stiles_selinv_workspace_bytes(const stiles_layout* lay) { return lay ? WS_ALIGN + sws_bytes(*lay) : 0; }

int stiles_pack(const double* ab, const double* arrow_rows, const double* corner, double* tiles,
                int64_t n, int64_t bandwidth, int64_t arrow, int32_t tile, void* stream) {
    stiles_layout lay;
    int rc = make_layout(n, bandwidth, arrow, tile, &lay);
    if (rc) return rc - 4;
    if (!ab) return -1;
    if (arrow > 0 && !arrow_rows) return -2;
    if (arrow > 0 && !corner) return -3;
    if (!tiles) return -4;
    Lay L = to_dev(lay);
    const int nab = arrow_blocks(L.ap);
    LAUNCH(STILES_TK_OTHER, k_pack, dim3((unsigned)(L.nt * (int64_t)(L.bt + 1) + L.nt + nab * nab)), dim3(NT), 0, S_(stream),
           ab, arrow_rows, corner, tiles, L);
    return 0;
}

int stiles_factor(const double* A, double* Lm, int64_t n, int64_t bandwidth, int64_t arrow, int32_t tile,
                  double* logdet, int32_t* info, void* workspace, size_t workspace_bytes, void* stream) {
    stiles_layout lay;
    int rc = make_layout(n, bandwidth, arrow, tile, &lay);
    if (rc) return rc - 2;
    if (!A) return -1;
    if (!Lm) return -2;
    if (!logdet) return -7;
    if (!info) return -8;
    if (!workspace || workspace_bytes < stiles_factor_workspace_bytes(&lay)) return -9;
    hipStream_t st = S_(stream);
    Lay L = to_dev(lay);
    const FactorWs f = factor_ws(L, ws_base(workspace));
    DevInfo di;
    if (dev_info(&di)) return STILES_EHIP;
    const FacCtx x = fac_ctx(L, Lm, f.Yd, f.flags);
    const int64_t ntask = fac_tasks(x), nticket = fac_chains(x) + ntask;
    if (nticket > 0x7fffffff) return -3;
    Sched sc;
    sc.ticket = f.ticket;
    sc.err = f.err;
    sc.spin_limit = spin_limit_ticks(di);
    sc.withhold = debug_withhold();

    if (A != Lm) {
        hipEvent_t tm = tm_begin(st);
        HIPCHK(hipMemcpyAsync(Lm, A, sizeof(double) * (size_t)L.total, hipMemcpyDeviceToDevice, st));
        tm_end(tm, STILES_TK_OTHER, st);
    }
    LAUNCH(STILES_TK_OTHER, k_factor_setup, dim3(grid_for(fac_ints(L) + fac_ints(corner_lay(L)))), dim3(NT), 0, st, L, f);
    LAUNCH(STILES_TK_FACTOR, fac_wide(Lm) ? k_factor_all<FAC_WIDE> : k_factor_all<FAC_NARROW>,
           dim3((unsigned)std::min<int64_t>(nticket, fac_grid(x, 2 * di.cus))), dim3(FAC_NT), 0, st, x, (int)ntask, sc, f.winfo);
    LAUNCH(STILES_TK_OTHER, k_factor_tail, dim3((unsigned)factor_tail_blocks(L)), dim3(NT), 0, st, Lm, L, f.ldp, f.Tc);
    if (L.ap > 0) {
        const FacCtx xc = corner_ctx(L, f);
        sc.ticket = f.cticket;
        sc.withhold = -1;
        LAUNCH(STILES_TK_POTRF, k_factor_all<FAC_WIDE>, dim3((unsigned)corner_grid(L)), dim3(FAC_NT), 0, st, xc, (int)fac_tasks(xc), sc,
               f.winfo);
        LAUNCH(STILES_TK_OTHER, k_corner_out, dim3((unsigned)corner_out_blocks(L)), dim3(NT), 0, st, Lm, L,
               (const double*)f.Tc, f.ldp, (const int*)f.winfo, (const int*)f.err, logdet, (int*)info);
        return 0;
    }
    LAUNCH(STILES_TK_OTHER, k_factor_final, dim3(1), dim3(64), 0, st, (const double*)f.ldp, factor_nparts(L),
           (const int*)f.winfo, (const int*)f.err, logdet, (int*)info);
    return 0;
}

// Selected inverse on the tile columns J >= jf (and the corner): Phase 1 of
// these columns, Phase 2 groups N-1 .. jf.  jf = 0 is the whole pattern.
static int selinv_impl(const double* Lm, double* S, const stiles_layout& lay, int64_t jf, int32_t* info,
                       void* workspace, hipStream_t st) {
    Lay L = to_dev(lay);
    const SelinvWs v = selinv_ws(L, ws_base(workspace));
    const int nb64 = L.b / 64, nab = arrow_blocks(L.ap);
    int64_t ntasks = 0;
    for (int64_t J = jf; J < L.nt; ++J) ntasks += p2_group_tasks(L, J, jf);
    if (ntasks > 0x7fffffff) return -3;
    const int64_t j1 = std::min<int64_t>(jf, L.nt - 1);

    LAUNCH(STILES_TK_OTHER, k_selinv_setup, dim3((unsigned)selinv_setup_grid(L)), dim3(NT), 0, st, L, S, v.flags, v.ticket,
           v.err, v.winfo);
    // Phase 1
    LAUNCH(STILES_TK_PHASE1, k_trtri_all, dim3((unsigned)(trtri_blocks(L) - j1 * trtri_per(L))), dim3(NT), 0, st, Lm, v.W, L, v.winfo,
           j1);
    {
        const int64_t g = (L.nt - j1) * (int64_t)(L.bt * nb64 + nab) * nb64;
        if (g > 0) {
            LAUNCH(STILES_TK_PHASE1, k_trmm_all, dim3((unsigned)g), dim3(NT), 0, st, Lm, v.W, L, j1);
        }
    }
    {
        const int64_t g = lauum_blocks(L, j1);
        LAUNCH(STILES_TK_PHASE1, k_lauum_all, dim3((unsigned)g), dim3(NT), 0, st, (const double*)v.W, S, L, j1);
    }
    // Phase 2, bottom-right to top-left, one persistent launch
    DevInfo di;
    if (dev_info(&di)) return STILES_EHIP;
    const P2 p = make_p2(S, L, v.W, L, v.flags, (int)ntasks, jf);
    Sched sc;
    sc.ticket = v.ticket;
    sc.err = v.err;
    sc.spin_limit = spin_limit_ticks(di);
    sc.withhold = debug_withhold();
    if (ntasks > 0) {
        const int grid = (int)std::min<int64_t>(ntasks, P2Cfg<8>::WG_PER_CU * (int64_t)di.cus);
        LAUNCH(STILES_TK_PHASE2, k_phase2, dim3(grid), dim3(P2Cfg<8>::NTH), 0, st, p, sc);
    }
    LAUNCH(STILES_TK_OTHER, k_selinv_final, dim3(1), dim3(64), 0, st, (const int*)v.winfo, (const int*)v.err,
           (int*)info);
    return 0;
}

int stiles_selinv(const double* Lm, double* S, int64_t n, int64_t bandwidth, int64_t arrow, int32_t tile,
                  int32_t* info, void* workspace, size_t workspace_bytes, void* stream) {
    stiles_layout lay;
    int rc = make_layout(n, bandwidth, arrow, tile, &lay);
    if (rc) return rc - 2;
    if (!Lm) return -1;
    if (!S || S == Lm) return -2;
    if (!info) return -7;
    if (!workspace || workspace_bytes < stiles_selinv_workspace_bytes(&lay)) return -8;
    return selinv_impl(Lm, S, lay, 0, info, workspace, S_(stream));
}

int stiles_selinv_range(const double* Lm, double* S, int64_t n, int64_t bandwidth, int64_t arrow, int32_t tile,
                        int64_t first_column, int32_t* info, void* workspace, size_t workspace_bytes, void* stream) {
    stiles_layout lay;
    int rc = make_layout(n, bandwidth, arrow, tile, &lay);
    if (rc) return rc - 2;
    if (!Lm) return -1;
    if (!S || S == Lm) return -2;
    if (first_column < 0 || first_column > lay.nt) return -7;
    if (!info) return -8;
    if (!workspace || workspace_bytes < stiles_selinv_workspace_bytes(&lay)) return -9;
    return selinv_impl(Lm, S, lay, first_column, info, workspace, S_(stream));
}

int stiles_gather(const double* Sigma, int64_t n, int64_t bandwidth, int64_t arrow, int32_t tile, const int64_t* ij,
                  int64_t count, double* out, void* stream) {
    stiles_layout lay;
    int rc = make_layout(n, bandwidth, arrow, tile, &lay);
    if (rc) return rc - 1;
    if (!Sigma) return -1;
    if (count < 0) return -7;
    if (count == 0) return 0;
    if (!ij) return -6;
    if (!out) return -8;
    LAUNCH(STILES_TK_OTHER, k_gather, dim3(grid_for(count)), dim3(NT), 0, S_(stream), Sigma, to_dev(lay), ij, count,
           out);
    return 0;
}

int stiles_selection_closure(int64_t n, int64_t bandwidth, int64_t arrow, int32_t tile, const int64_t* ij,
                             int64_t count, int32_t* inside, int64_t* first_column) {
    stiles_layout lay;
    int rc = make_layout(n, bandwidth, arrow, tile, &lay);
    if (rc) return rc;
    if (count < 0) return -6;
    if (count > 0 && !ij) return -5;
    if (!inside) return -7;
    if (!first_column) return -8;
    const int64_t b = lay.tile, nb = lay.nb;
    int32_t in = 1;
    int64_t first = lay.nt;
    for (int64_t k = 0; k < count; ++k) {
        const int64_t i = ij[2 * k], j = ij[2 * k + 1];
        const int64_t hi = i > j ? i : j, lo = i > j ? j : i;
        if (lo < 0 || hi >= n) return -5;
        // a band entry lies in L's tile pattern when its tile row is within
        // B tiles of its tile column; arrow rows and the corner always do
        if (hi < nb && hi / b - lo / b > lay.bt) in = 0;
        const int64_t col = lo < nb ? lo / b : lay.nt;
        if (col < first) first = col;
    }
    *inside = in;
    *first_column = first;
    return 0;
}

int stiles_mfma_peak(double* sink, int64_t sink_doubles, int32_t iters, double* flops, void* stream) {
    if (!flops) return -4;
    if (iters < 1) return -3;
    DevInfo di;
    if (dev_info(&di)) return STILES_EHIP;
    const int64_t blocks = 2 * (int64_t)di.cus;
    if (!sink || sink_doubles < blocks * NT) return -1;
    *flops = (double)blocks * (NT / 64) * (double)iters * PEAK_CHAINS * 2048.0;
    hipLaunchKernelGGL(k_mfma_peak, dim3((unsigned)blocks), dim3(NT), 0, S_(stream), sink, (int)iters);
    LAUNCHCHK();
    return 0;
}

size_t stiles_trace_workspace_bytes(void) { return sizeof(double) * TP_BLOCKS; }

// inverse workspace: the selected inverse's, Sigma in the dense layout, its
// Phase 2 counters; never less than a dense matrix beside the first, which
// callers may count on
size_t stiles_inverse_workspace_bytes(const stiles_layout* lay) {
    if (!lay) return 0;
    const Lay F = full_lay(to_dev(*lay));
    const size_t np = (size_t)(lay->nt * lay->tile + lay->arrow_ld);
    return WS_ALIGN + align256(sws_bytes(*lay)) +
           std::max(sizeof(double) * np * np, sizeof(double) * (size_t)F.total + sizeof(int) * (size_t)((F.bt + 2) * F.nt));
}

int stiles_inverse(const double* Lm, double* Ainv, int64_t n, int64_t bandwidth, int64_t arrow, int32_t tile,
                   int32_t* info, void* workspace, size_t workspace_bytes, void* stream) {
    stiles_layout lay;
    int rc = make_layout(n, bandwidth, arrow, tile, &lay);
    if (rc) return rc - 2;
    if (!Lm) return -1;
    if (!Ainv) return -2;
    if (!info) return -7;
    if (!workspace || workspace_bytes < stiles_inverse_workspace_bytes(&lay)) return -8;
    hipStream_t st = S_(stream);
    const Lay L = to_dev(lay), F = full_lay(L);
    const SelinvWs v = selinv_ws(L, ws_base(workspace));
    double* D = (double*)(ws_base(workspace) + align256(sws_bytes(lay)));
    int* cnt = (int*)(D + F.total);
    const int nb64 = L.b / 64, nab = arrow_blocks(L.ap);
    const int64_t ntasks = p2_total_tasks(F), n64 = (lay.n + 63) / 64;
    if (ntasks > 0x7fffffff || n64 * (n64 + 1) / 2 > 0x7fffffff) return -3;
    DevInfo di;
    if (dev_info(&di)) return STILES_EHIP;

    LAUNCH(STILES_TK_OTHER, k_selinv_setup, dim3(64), dim3(NT), 0, st, F, (double*)nullptr, cnt, v.ticket, v.err,
           v.winfo);
    // Phase 1: X_J, Lhat (as for stiles_selinv)
    LAUNCH(STILES_TK_PHASE1, k_trtri_all, dim3((unsigned)trtri_blocks(L)), dim3(NT), 0, st, Lm, v.W, L, v.winfo,
           (int64_t)0);
    {
        const int64_t g = L.nt * (int64_t)(L.bt * nb64 + nab) * nb64;
        if (g > 0) LAUNCH(STILES_TK_PHASE1, k_trmm_all, dim3((unsigned)g), dim3(NT), 0, st, Lm, v.W, L, (int64_t)0);
    }
    LAUNCH(STILES_TK_PHASE1, k_inv_lauum, dim3((unsigned)lauum_blocks(L, 0)), dim3(NT), 0, st, (const double*)v.W, L, D, F);
    Sched sc;
    sc.ticket = v.ticket;
    sc.err = v.err;
    sc.spin_limit = spin_limit_ticks(di);
    sc.withhold = -1;
    const int grid = (int)std::min<int64_t>(ntasks, P2Cfg<8>::WG_PER_CU * (int64_t)di.cus);
    LAUNCH(STILES_TK_PHASE2, k_phase2, dim3(grid), dim3(P2Cfg<8>::NTH), 0, st, make_p2(D, F, v.W, L, cnt, (int)ntasks, 0), sc);
    LAUNCH(STILES_TK_OTHER, k_inv_compact, dim3((unsigned)(n64 * (n64 + 1) / 2)), dim3(NT), 0, st, (const double*)D, F,
           Ainv);
    LAUNCH(STILES_TK_OTHER, k_selinv_final, dim3(1), dim3(64), 0, st, (const int*)v.winfo, (const int*)v.err, (int*)info);
    return 0;
}

int stiles_trace_product(const double* Sigma, const double* B, int64_t n, int64_t bandwidth, int64_t arrow,
                         int32_t tile, double* out, void* workspace, size_t workspace_bytes, void* stream) {
    stiles_layout lay;
    int rc = make_layout(n, bandwidth, arrow, tile, &lay);
    if (rc) return rc - 2;
    if (!Sigma) return -1;
    if (!B) return -2;
    if (!out) return -7;
    if (!workspace || workspace_bytes < stiles_trace_workspace_bytes()) return -8;
    hipStream_t st = S_(stream);
    const Lay L = to_dev(lay);
    double* part = (double*)workspace;
    LAUNCH(STILES_TK_OTHER, k_trace_part, dim3(TP_BLOCKS), dim3(NT), 0, st, Sigma, B, L, part);
    LAUNCH(STILES_TK_OTHER, k_trace_final, dim3(1), dim3(64), 0, st, (const double*)part, out);
    return 0;
}

size_t stiles_batch_workspace_bytes(const stiles_batch_item* items, int32_t count) {
    if (!items || count < 1) return 0;
    BPlan pl;
    if (batch_plan(items, count, false, pl)) return 0;
    return pl.total;
}

// Host side of both batched calls: the matrix table (and the segment tables
// appended to `segs`) go to the table area of the workspace in one copy.
// Pinned host buffers for the table uploads, kept for the life of the
// process.  A buffer is handed out again only once the event recorded after
// its copy has completed, so calls on several streams at once (concurrent
// serving lanes) never overwrite a table that is still being copied.
struct PinnedBuf {
    char* p;
    size_t cap;
    hipEvent_t done;
};
static std::mutex g_pmu;
static std::vector<PinnedBuf> g_pin;
#define PIN_MAX_BUFS 16

// Host bytes -> device, through a pinned buffer, on stream st.
static int pinned_upload(void* dst, const void* src, size_t n, hipStream_t st) {
    std::lock_guard<std::mutex> lk(g_pmu);
    PinnedBuf* b = nullptr;
    for (auto& x : g_pin)
        if (x.cap >= n && hipEventQuery(x.done) == hipSuccess) {
            b = &x;
            break;
        }
    if (!b && g_pin.size() < PIN_MAX_BUFS) {
        PinnedBuf x;
        x.cap = std::max<size_t>(n, 1 << 16);
        HIPCHK(hipHostMalloc((void**)&x.p, x.cap, hipHostMallocDefault));
        if (hipEventCreateWithFlags(&x.done, hipEventDisableTiming) != hipSuccess) {
            (void)hipHostFree(x.p);
            return STILES_EHIP;
        }
        g_pin.push_back(x);
        b = &g_pin.back();
    }
    if (!b) {
        // every buffer busy: wait for the first one large enough, else grow it
        b = &g_pin[0];
        for (auto& x : g_pin)
            if (x.cap >= n) {
                b = &x;
                break;
            }
        HIPCHK(hipEventSynchronize(b->done));
        if (b->cap < n) {
            HIPCHK(hipHostFree(b->p));
            b->cap = n;
            HIPCHK(hipHostMalloc((void**)&b->p, b->cap, hipHostMallocDefault));
        }
    }
    memcpy(b->p, src, n);
    HIPCHK(hipMemcpyAsync(dst, b->p, n, hipMemcpyHostToDevice, st));
    HIPCHK(hipEventRecord(b->done, st));
    return 0;
}

static int batch_upload(const std::vector<BInst>& bi, const std::vector<BSeg>& segs, char* ws, hipStream_t st) {
    const size_t o1 = align256(sizeof(BInst) * bi.size());
    std::vector<char> h(o1 + sizeof(BSeg) * segs.size());
    memcpy(h.data(), bi.data(), sizeof(BInst) * bi.size());
    memcpy(h.data() + o1, segs.data(), sizeof(BSeg) * segs.size());
    return pinned_upload(ws, h.data(), h.size(), st);
}

// What a batched call does: upload its tables (host -> workspace), enqueue its
// kernels
// (device work only, reading the tables; what a HIP graph can capture), or both.
#define BATCH_UPLOAD 1
#define BATCH_LAUNCH 2
static int factor_batched_impl(const stiles_batch_item* items, int32_t count, void* workspace,
                               size_t workspace_bytes, void* stream, int mode) {
    if (!items) return -1;
    if (count < 1) return -2;
    BPlan pl;
    if (batch_plan(items, count, false, pl)) return -1;
    if (!workspace) return -3;
    if (workspace_bytes < pl.total) return -4;
    hipStream_t st = S_(stream);
    DevInfo di;
    if (dev_info(&di)) return STILES_EHIP;
    char* ws = ws_base(workspace);
    std::vector<BInst> bi(count);
    for (int k = 0; k < count; ++k) {
        BInst& I = bi[k];
        memset(&I, 0, sizeof(I));
        I.L = to_dev(pl.lay[k]);
        I.A = items[k].A;
        I.Lm = items[k].L;
        I.S = items[k].Sigma;
        I.logdet = items[k].logdet;
        I.info = items[k].info;
        I.ws = ws + pl.off[k];
        I.nparts = factor_nparts(I.L);
        const FacCtx x = fac_ctx(I.L, nullptr, nullptr, nullptr);
        const int64_t n = fac_tasks(x), nticket = fac_chains(x) + n;
        if (nticket > 0x7fffffff) return -1;
        I.fac_ntask = (int)n;
        I.fac_nticket = (int)nticket;
    }
    const size_t seg0 = align256(sizeof(BInst) * (size_t)count);
    const size_t int0 = seg0 + align256(sizeof(BSeg) * batch_nseg(count));
    std::vector<BSeg> segs;
    SegTab t;
    t.start(segs.size());
    for (int k = 0; k < count; ++k) t.add(segs, k, factor_tail_blocks(bi[k].L));
    struct Launch { size_t at; int n, grid; };
    auto close = [&](Launch& l) { l.at = t.begin; l.grid = t.grid; l.n = t.finish(segs); };
    Launch tail, corner, corner_back;
    close(tail);
    t.start(segs.size());
    for (int k = 0; k < count; ++k)
        if (bi[k].L.ap > 0) t.add(segs, k, corner_grid(bi[k].L));
    close(corner);
    t.start(segs.size());
    for (int k = 0; k < count; ++k)
        if (bi[k].L.ap > 0) t.add(segs, k, corner_out_blocks(bi[k].L));
    close(corner_back);
    // the factor: the resident workgroups shared in proportion to the tickets,
    // at least two per matrix (one when it has only its chain)
    std::vector<Launch> fac;
    for (int k0 = 0; k0 < count; k0 += KB_SLICE) {
        const int k1 = std::min(count, k0 + KB_SLICE);
        int64_t sum = 0;
        for (int k = k0; k < k1; ++k) sum += bi[k].fac_nticket;
        t.start(segs.size());
        for (int k = k0; k < k1; ++k) {
            const int64_t n = bi[k].fac_nticket, want = 2 * (int64_t)di.cus * n / sum;
            t.add(segs, k, (int)std::min<int64_t>(n, std::max<int64_t>(2, want)));
        }
        Launch l;
        close(l);
        fac.push_back(l);
    }
    if (mode & BATCH_UPLOAD) {
        const int rc = batch_upload(bi, segs, ws, st);
        if (rc) return rc;
    }
    if (!(mode & BATCH_LAUNCH)) return 0;
    const BInst* dbi = (const BInst*)ws;
    const BSeg* dseg = (const BSeg*)(ws + seg0);
    int* dint = (int*)(ws + int0);
    const int64_t spin = spin_limit_ticks(di);

    LAUNCH(STILES_TK_OTHER, k_zero_ints, dim3(1), dim3(NT), 0, st, dint, (int64_t)1);
    for (int k = 0; k < count; ++k) {
        if (bi[k].A == bi[k].Lm) continue;
        hipEvent_t tm = tm_begin(st);
        HIPCHK(hipMemcpyAsync(bi[k].Lm, bi[k].A, sizeof(double) * (size_t)bi[k].L.total, hipMemcpyDeviceToDevice, st));
        tm_end(tm, STILES_TK_OTHER, st);
    }
    LAUNCH(STILES_TK_OTHER, kb_factor_setup, dim3((unsigned)(8 * count)), dim3(NT), 0, st, dbi);
    auto args = [&](const Launch& l) { return BArgs{dbi, dseg + l.at, l.n, spin}; };
    bool wide = true;   // every L
    for (int k = 0; k < count; ++k) wide = wide && fac_wide(bi[k].Lm);
    for (size_t q = 0; q < fac.size(); ++q)
        LAUNCH(STILES_TK_FACTOR, wide ? kb_factor<FAC_WIDE> : kb_factor<FAC_NARROW>, dim3((unsigned)fac[q].grid), dim3(FAC_NT), 0, st, args(fac[q]),
               (int)q * KB_SLICE, std::min<int>(count, ((int)q + 1) * KB_SLICE), dint);
    LAUNCH(STILES_TK_OTHER, kb_factor_tail, dim3((unsigned)tail.grid), dim3(NT), 0, st, args(tail));
    if (corner.grid > 0) {
        LAUNCH(STILES_TK_POTRF, kb_corner, dim3((unsigned)corner.grid), dim3(FAC_NT), 0, st, args(corner), dint);
        LAUNCH(STILES_TK_OTHER, kb_corner_out, dim3((unsigned)corner_back.grid), dim3(NT), 0, st, args(corner_back));
    }
    LAUNCH(STILES_TK_OTHER, kb_factor_final, dim3(count), dim3(64), 0, st, dbi, (const int*)dint);
    return 0;
}

static int selinv_batched_impl(const stiles_batch_item* items, int32_t count, void* workspace,
                               size_t workspace_bytes, void* stream, int mode) {
    if (!items) return -1;
    if (count < 1) return -2;
    BPlan pl;
    if (batch_plan(items, count, true, pl)) return -1;
    if (!workspace) return -3;
    if (workspace_bytes < pl.total) return -4;
    hipStream_t st = S_(stream);
    DevInfo di;
    if (dev_info(&di)) return STILES_EHIP;
    char* ws = ws_base(workspace);
    char* tab = ws + pl.table_f;   // this call's table area
    std::vector<BInst> bi(count);
    int64_t sum_tasks = 0;
    for (int k = 0; k < count; ++k) {
        BInst& I = bi[k];
        memset(&I, 0, sizeof(I));
        I.L = to_dev(pl.lay[k]);
        I.A = items[k].A;
        I.Lm = items[k].L;
        I.S = items[k].Sigma;
        I.logdet = items[k].logdet;
        I.info = items[k].info;
        I.ws = ws + pl.off[k];
        I.p2_tasks = (int)p2_total_tasks(I.L);
        sum_tasks += I.p2_tasks;
    }
    const size_t seg0 = align256(sizeof(BInst) * (size_t)count);
    std::vector<BSeg> segs;
    SegTab t;
    struct Launch { size_t at; int n, grid; };
    auto close = [&](Launch& l) { l.at = t.begin; l.grid = t.grid; l.n = t.finish(segs); };
    Launch zu, tr, tm, la, p2;
    t.start(segs.size());
    for (int k = 0; k < count; ++k) t.add(segs, k, std::min(selinv_setup_grid(bi[k].L), 256));
    close(zu);
    t.start(segs.size());
    for (int k = 0; k < count; ++k) t.add(segs, k, trtri_blocks(bi[k].L));
    close(tr);
    t.start(segs.size());
    for (int k = 0; k < count; ++k) {
        const Lay& L = bi[k].L;
        const int nb64 = L.b / 64;
        t.add(segs, k, (int)(L.nt * (int64_t)(L.bt * nb64 + arrow_blocks(L.ap)) * nb64));
    }
    close(tm);
    t.start(segs.size());
    for (int k = 0; k < count; ++k) t.add(segs, k, (int)lauum_blocks(bi[k].L, 0));
    close(la);
    // Eight wavefronts per workgroup (one per CU) when the matrices' tile
    // columns together hold few tasks, so that their length counts, else four
    // (two per CU).  Measured, eight against four: 170 to 360 tasks 0.36 / 0.42
    // and 1.60 / 2.12 ms, 8 served matrices 8.5 / 9.0, 860 tasks the same, 830
    // with longer sums 23.2 / 17.9, 1,730 1.76 / 1.39.
    double column = 0.0;
    for (int k = 0; k < count; ++k) column += (double)bi[k].p2_tasks / (double)bi[k].L.nt;
    const bool wide = column <= P2_WIDE_TASKS;
    // Phase 2: the resident workgroups shared in proportion to the work, at
    // least one per matrix
    t.start(segs.size());
    {
        double work = 0.0;
        for (int k = 0; k < count; ++k) work += p2_work(bi[k].L, bi[k].p2_tasks);
        const int64_t total = std::min<int64_t>(sum_tasks, (wide ? P2Cfg<8>::WG_PER_CU : P2Cfg<4>::WG_PER_CU) * (int64_t)di.cus);
        for (int k = 0; k < count; ++k) {
            const int64_t want = (int64_t)((double)total * p2_work(bi[k].L, bi[k].p2_tasks) / work);
            t.add(segs, k, (int)std::max<int64_t>(1, std::min<int64_t>(bi[k].p2_tasks, want)));
        }
    }
    close(p2);
    if (mode & BATCH_UPLOAD) {
        const int rc = batch_upload(bi, segs, tab, st);
        if (rc) return rc;
    }
    if (!(mode & BATCH_LAUNCH)) return 0;
    const BInst* dbi = (const BInst*)tab;
    const BSeg* dseg = (const BSeg*)(tab + seg0);
    const int64_t spin = spin_limit_ticks(di);
    auto args = [&](const Launch& l) { return BArgs{dbi, dseg + l.at, l.n, spin}; };

    LAUNCH(STILES_TK_OTHER, kb_selinv_setup, dim3((unsigned)zu.grid), dim3(NT), 0, st, args(zu));
    LAUNCH(STILES_TK_PHASE1, kb_trtri, dim3((unsigned)tr.grid), dim3(NT), 0, st, args(tr));
    if (tm.grid > 0) LAUNCH(STILES_TK_PHASE1, kb_trmm, dim3((unsigned)tm.grid), dim3(NT), 0, st, args(tm));
    LAUNCH(STILES_TK_PHASE1, kb_lauum, dim3((unsigned)la.grid), dim3(NT), 0, st, args(la));
    if (wide) LAUNCH(STILES_TK_PHASE2, kb_phase2<8>, dim3((unsigned)p2.grid), dim3(P2Cfg<8>::NTH), 0, st, args(p2), (int)count);
    else LAUNCH(STILES_TK_PHASE2, kb_phase2<4>, dim3((unsigned)p2.grid), dim3(P2Cfg<4>::NTH), 0, st, args(p2), (int)count);
    LAUNCH(STILES_TK_OTHER, kb_selinv_final, dim3(count), dim3(64), 0, st, dbi);
    return 0;
}

int stiles_factor_batched(const stiles_batch_item* items, int32_t count, void* workspace, size_t workspace_bytes,
                          void* stream) {
    return factor_batched_impl(items, count, workspace, workspace_bytes, stream, BATCH_UPLOAD | BATCH_LAUNCH);
}

int stiles_selinv_batched(const stiles_batch_item* items, int32_t count, void* workspace, size_t workspace_bytes,
                          void* stream) {
    return selinv_batched_impl(items, count, workspace, workspace_bytes, stream, BATCH_UPLOAD | BATCH_LAUNCH);
}

int stiles_batch_upload(const stiles_batch_item* items, int32_t count, void* workspace, size_t workspace_bytes,
                        void* stream) {
    const int rc = factor_batched_impl(items, count, workspace, workspace_bytes, stream, BATCH_UPLOAD);
    if (rc) return rc;
    return selinv_batched_impl(items, count, workspace, workspace_bytes, stream, BATCH_UPLOAD);
}

int stiles_factor_batched_enqueue(const stiles_batch_item* items, int32_t count, void* workspace,
                                  size_t workspace_bytes, void* stream) {
    return factor_batched_impl(items, count, workspace, workspace_bytes, stream, BATCH_LAUNCH);
}

int stiles_selinv_batched_enqueue(const stiles_batch_item* items, int32_t count, void* workspace,
                                  size_t workspace_bytes, void* stream) {
    return selinv_batched_impl(items, count, workspace, workspace_bytes, stream, BATCH_LAUNCH);
}

}  // extern "C"
