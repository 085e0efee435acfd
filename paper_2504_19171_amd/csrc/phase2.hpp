// Phase 2 of the selected inversion as one persistent launch.
//
// Tile column J needs the off-diagonal tiles S(J) x S(J) of Sigma, where
// S(J) = band tiles J+1..J+s and the arrow:
//   Sigma_{i,J} = -sum_{k in S(J)} Sigma_{i,k} Lhat_{k,J}              i in S(J)
//   Sigma_JJ = X_J^T X_J - sum_{i in S(J)} Lhat_{i,J}^T Sigma_{i,J}
// Every block is formed by one task, which takes its sum in the order in which
// the operands become final, as their counters come up, and writes the block
// once:
//   FAR : a 64 x 64 block of a row tile J+2..J+s or of the arrow.  A 32 x 32
//     quadrant per wavefront over the whole sum, the operands staged through
//     LDS for all four: the arrow's term first, then k = J+s down to J+1, so
//     only the last products wait for column J+1.
//   ROW : a 32 x 32 block of row tile J+1, the sum spread over the
//     wavefronts: k = J+2.. and the arrow (column J+1's off-diagonal tiles),
//     then k = J+1 (its diagonal tile).
//   DIAG: a 32 x 32 block of the lower triangle of Sigma_JJ, likewise: the
//     arrow and rows J+3.., then J+2 and J+1; mirrored.
// What bounds it: the chain DIAG(J+1) -> ROW(J) -> DIAG(J) (and FAR(J+1) ->
// FAR(J)) where there are few blocks, the matrix cores where there are many.
// The sums are not cut into tasks of their own, because the resident
// workgroups hold the next tickets whether these can run or not: with 32 x 32
// tasks for the early and late part of each sum (940 a column at tile 256,
// w 1,024) they covered half a tile column; these are 156.  Before and after,
// ms: nb 100,000 w 1,024 a 100 tile 256 16.8 -> 9.5 (24 us a column); w 2,001
// 39.3 -> 20.0; nb 15,999 w 553 a 413 tile 128 4.8 -> 2.0; nb 31,987 w 32 a 57
// tile 64 5.6 -> 3.9; 64 matrices of tile 64 49.6 -> 26.0.
// Tickets: FAR(N-1), then groups J = N-1 .. 0, each FAR(J-1) but for row tile
// J+1, ROW(J), the rest of FAR(J-1), DIAG(J); a task depends only on earlier
// tickets.  FAR(J-1) needs nothing of DIAG(J), and starts well before (with
// FAR(J), ROW(J), DIAG(J) in turn w 2,001 took 25.6 ms against 20.9).  Counters: finished tasks per tile, cnt[J (bt + 2) + d]
// for tile (J+d, J), d <= bt, and d = bt + 1 for the arrow tile.
#pragma once
#include "common.hpp"
#include "persist.hpp"
#include "wave_gemm.hpp"
#include "factor.hpp"

#define ARW (-1)   // "the arrow" in place of a band tile offset

enum { P2_FAR = 0, P2_ROW, P2_DIAG };

struct P2 {
    double* S;
    const double* W;
    Lay L;      // of Sigma
    // of W: its tile half-bandwidth and arrow offset.  The same as Sigma's for
    // the selected inverse; for the whole inverse Sigma has every tile below
    // the diagonal, and the sums still run over W's band and arrow only.
    int btw;
    int64_t warrow;
    int* cnt;
    int ntasks;
    // rows of the last band tile (J + bt) that Lhat's band reaches, to 32
    int klast;
    int jf;   // the first tile column wanted
    // groups are taken in the order J = N-1-q, q = 0, 1, ...; from q = q0 on
    // every group but the last holds g_tasks tasks, and group q0 starts at
    // ticket off_q0, so a ticket's group is found in closed form
    int q0, off_q0, g_tasks;

    __host__ __device__ int sw(int64_t J) const { return (int)(L.nt - 1 - J < btw ? L.nt - 1 - J : btw); }
    __host__ __device__ int64_t wband(int64_t J, int e) const { return (J * (int64_t)(btw + 1) + e) * L.b * L.b; }
    __host__ __device__ int64_t war(int64_t J) const { return warrow + J * (int64_t)L.ap * L.b; }
};

__host__ __device__ inline int p2_ctr(const Lay& L) { return L.bt + 2; }   // counters per tile column
__host__ __device__ inline int p2_arw(const Lay& L) { return L.bt + 1; }
__host__ __device__ inline int p2_far_tasks(const Lay& L, int64_t J) {
    const int nb64 = L.b / 64, s = L.s(J);
    return ((s > 1 ? s - 1 : 0) * nb64 + arrow_blocks(L.ap)) * nb64;
}
__host__ __device__ inline int p2_row_tasks(const Lay& L, int64_t J) {
    return L.s(J) >= 1 ? (L.b / 32) * (L.b / 32) : 0;
}
__host__ __device__ inline int p2_diag_tasks(const Lay& L) { return (L.b / 32) * (L.b / 32 + 1) / 2; }
// FAR tasks of row tile J + 2, the last ones of a column
__host__ __device__ inline int p2_far2_tasks(const Lay& L, int64_t J) {
    return L.s(J) > 1 ? (L.b / 64) * (L.b / 64) : 0;
}
// Tasks of group J (jf: the first tile column wanted).
__host__ __device__ inline int p2_group_tasks(const Lay& L, int64_t J, int64_t jf) {
    return (J == L.nt - 1 ? p2_far_tasks(L, J) : 0) + (J > jf ? p2_far_tasks(L, J - 1) : 0) + p2_row_tasks(L, J) +
           p2_diag_tasks(L);
}
// Tasks before group q <= max(bt, 1), none of these the last: one more row tile
// in each than in the one before.
__host__ __device__ inline int64_t p2_base(const Lay& L, int64_t q) {
    if (q == 0) return 0;
    const int64_t nb64 = L.b / 64, nab = arrow_blocks(L.ap);
    return nb64 * nb64 * (q * (q - 1) / 2) + q * (nab * nb64 + p2_diag_tasks(L)) + (q - 1) * 4 * nb64 * nb64 + nab * nb64;
}
// Tasks that make tile offset d (or ARW) of a column final.
__device__ inline int p2_target(const Lay& L, int d) {
    const int nb64 = L.b / 64;
    if (d == 0) return p2_diag_tasks(L);
    if (d == 1) return 4 * nb64 * nb64;
    return (d == ARW ? arrow_blocks(L.ap) : nb64) * nb64;
}
__device__ inline const int* p2_counter(const P2& p, int64_t J, int d) {
    return p.cnt + J * p2_ctr(p.L) + (d == ARW ? p2_arw(p.L) : d);
}

__device__ inline void p2_setup_body(const Lay& L, int* cnt, int* ticket, int* err, int* info, int bid, int nblk) {
    const int64_t n = (int64_t)p2_ctr(L) * L.nt;
    for (int64_t i = threadIdx.x + (int64_t)bid * blockDim.x; i < n; i += (int64_t)nblk * blockDim.x) cnt[i] = 0;
    if (bid == 0 && threadIdx.x == 0) {
        *ticket = 0;
        *err = 0;
        *info = 0;
    }
}

// Operand A = Sigma restricted to a block of rows and a tile of k:
// rows = block rbl (of rb rows) of tile J+d (d >= 1) or of the arrow (ARW);
// k = tile J+e (e >= 1) or the arrow.
__device__ inline void p2_sigma_rows(const Lay& L, const double* S, int64_t J, int d, int rbl, int rb, int e,
                                     const double*& a, int64_t& lda, int& ta, int& av) {
    av = rb;
    if (d != ARW && e != ARW) {
        if (d > e) { a = S + L.band(J + e, d - e) + rbl * rb; lda = L.b; ta = 0; }
        else if (d == e) { a = S + L.band(J + d, 0) + rbl * rb; lda = L.b; ta = 0; }
        else { a = S + L.band(J + d, e - d) + (int64_t)rbl * rb * L.b; lda = L.b; ta = 1; }
    } else if (d != ARW) {
        a = S + L.arrow(J + d) + (int64_t)rbl * rb * L.ap; lda = L.ap; ta = 1;
    } else {
        av = imin_(rb, L.ap - rbl * rb);
        lda = L.ap; ta = 0;
        a = (e != ARW) ? S + L.arrow(J + e) + rbl * rb : S + L.corner() + rbl * rb;
    }
}

// The counter of Sigma_{J+d, J+e} (the corner, d and e both ARW, is final).
__device__ inline void p2_sigma_dep(const P2& p, int64_t J, int d, int e, const int*& f, int& target) {
    int64_t c;
    int o;
    if (d == ARW && e == ARW) { f = p.cnt; target = 0; return; }
    if (d == ARW) { c = J + e; o = ARW; }
    else if (e == ARW) { c = J + d; o = ARW; }
    else { c = J + imin_(d, e); o = imax_(d, e) - imin_(d, e); }
    f = p2_counter(p, c, o);
    target = p2_target(p.L, o);
}

// How many of the n operands q = 0 .. n-1 (dep(q, counter, target)) are ready,
// from the first on; waits for `need` of them.  At most 64 are looked at.
// 0: the kernel must stop.  meanwhile() is called once by every wavefront, by
// the one that looks after its first look; its loads may be in flight on return.
template <class F, class G>
__device__ inline int p2_ready(const Sched& sc, int n, int need, int* sh, F&& dep, G&& meanwhile) {
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0) {
        const int lane = threadIdx.x & 63, m = imin_(n, 64);
        const int* f;
        int target;
        dep(imin_(lane, m - 1), f, target);
        int k = 0;
        int64_t t0 = -1;
        for (unsigned polls = 0;; ++polls) {
            const uint64_t b = __ballot(ld_coh_i(f) >= target);
            k = ~b == 0 ? m : imin_(m, (int)__builtin_ctzll(~b));
            if (polls == 0) meanwhile();
            if (k >= need) break;
            if (t0 < 0) t0 = wall_clock64();
            if ((polls & 15) == 15) {
                bool stop = __builtin_amdgcn_readfirstlane(ld_coh_i(sc.err)) != 0;
                if (!stop && wall_clock64() - t0 > sc.spin_limit) {
                    set_error_once(sc.err, STILES_ETIMEOUT);
                    stop = true;
                }
                if (stop) { k = 0; break; }
            }
            __builtin_amdgcn_s_sleep(2);   // (1: 9.50 against 9.39 ms at w 1,024; two looks in flight: 9.75)
        }
        if (lane == 0) fac_lds_set(sh, k);
    } else {
        meanwhile();
    }
    // (not __syncthreads, which would wait for meanwhile()'s loads)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    return __builtin_amdgcn_readfirstlane(fac_lds_get(sh));
}
// All n of them, any number.
template <class F, class G>
__device__ inline bool p2_all_ready(const Sched& sc, int n, int* sh, F&& dep, G&& meanwhile) {
    for (int q = 0; q < n; q += 64) {
        const int m = imin_(n - q, 64);
        const int k = p2_ready(sc, m, m, sh, [&](int e, const int*& f, int& t) { dep(q + e, f, t); },
                               [&]() { if (q == 0) meanwhile(); });
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // *sh has been read by all
        if (k == 0) return false;
    }
    return true;
}

// NW wavefronts per workgroup: 8 (one workgroup per CU) for a single matrix,
// where the length of a task counts (four, two per CU: w 1,024 17.2 ms against
// 11.5, w 2,001 29.9 against 27.5), 4 (two per CU) for a batch, where one
// workgroup computes while the other waits, loads or stores.  The sums are the
// same bit for bit.  LDS: the staging of FAR (four stages), of ROW and DIAG
// (the wavefronts' areas, which wave_reduce reuses), and the reduced block.
template <int NW>
struct P2Cfg {
    static constexpr int NTH = 64 * NW;
    static constexpr int STAGE = NW * (WG_WAVE > WR_DOUBLES ? WG_WAVE : WR_DOUBLES);
    static constexpr int SMEM = STAGE + WR_DOUBLES;
    static constexpr int WG_PER_CU = 8 / NW;
};

// ---------------------------------------------------------------------------
// FAR
// ---------------------------------------------------------------------------
#define FAR_STAGES 4
// One term of a FAR sum: Sigma(x, k) = ta ? a[k + x lda] : a[x + k lda], x < av
// (rows past av repeat existing ones), Lhat(k, j) = b[k + j ldb], k < K.
struct FarSeg {
    const double* a;
    const double* b;
    int lda, ldb, ta, av, K;
};
#define FAR_OPND (64 * 16)          // doubles of one operand in a stage
#define FAR_STAGE (2 * FAR_OPND)
// 16 k of one operand go straight into LDS by four wavefronts (v: 0 .. 3), two
// kilobyte loads each.  Element (x, k) of an operand contiguous along x lies at
// [k * 64 + (x ^ 16 (k / 2 % 4))] (one along k: see wg_lane).  far_lanes: where
// in the operand this lane's loads begin.
__device__ __forceinline__ void far_lanes(int ld, int contig_x, int av, int v, uint32_t (&o)[2]) {
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = 2 * v + u;   // the load's kilobyte
        if (contig_x) {
            const int k = 2 * i + (l >> 5), x = (2 * (l & 31)) ^ (16 * (i & 3));
            o[u] = (uint32_t)(imin_(x, av - 2) + k * ld);
        } else {
            o[u] = wg_lane(ld, i);
        }
    }
}
template <int COH>
__device__ __forceinline__ void far_fetch(const double* b, const uint32_t (&o)[2], int v, double* st) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
        __builtin_amdgcn_global_load_lds((const void*)((const char*)b + (o[u] << 3)), (lds_void_t*)(st + 128 * (2 * v + u)), 16,
                                         0, COH ? 16 : 0);
}

// Wait until the oldest of this wavefront's stages (4 loads each) has landed,
// `later` stages issued after it.
__device__ __forceinline__ void far_landed(int later) {
    if (later >= 2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else if (later == 1) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The products of one stage; issue() in their midst (its arithmetic runs beside
// the matrix cores).
struct FarAddr {
    uint32_t x0, x1, k0, k1, b0, b1;   // operands in stage 0: Sigma along x, along k; Lhat (along k)
};
template <class F>
__device__ __forceinline__ void far_mma(dbl4 (&acc)[2][2], const FarAddr& f, int ta, uint32_t so, F&& issue) {
    wg2 a[2][2], b[2][2];
    if (ta) wg_read_kk(f.k0 + so, f.k1 + so, f.b0 + so, f.b1 + so, a, b);
    else wg_read_xk(f.x0 + so, f.x1 + so, f.b0 + so, f.b1 + so, a, b);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[j][m].x, a[i][m].x, acc[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[j][m].y, a[i][m].y, acc[i][j], 0, 0, 0);
        if (m == 0) issue();
    }
}

// acc += the terms q0 .. q1 - 1 (seg(q)), in steps of 32 k of a term: acc0 the
// first 16 of each, acc1 the others, if the term has them (NW = 8: wavefronts
// 0 .. 3 hold the one, 4 .. 7 the other, each set with its own stages and both
// as acc0).  acc[i][j]: rows 32 (v % 2) + 16 i, columns 32 (v / 2) + 16 j of
// the block for wavefront v of four, transposed on the matrix cores: element r
// is (row .. + l % 16, column .. + 4 r + l / 16), so that stores run down a
// column.  The workgroup's LDS holds nothing else while this runs; at the end
// some wavefronts may still be reading the last stage.
template <int NW, class F>
__device__ __forceinline__ void far_sum(dbl4 (&acc0)[2][2], dbl4 (&acc1)[2][2], int q0, int q1, double* smem, F&& seg) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), v = w & 3, half = w >> 2;
    const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
    const int rx = 32 * (v & 1) + li, cx = 32 * (v >> 1) + li;
    double* ring = smem + half * (FAR_STAGES * FAR_STAGE);
    const uint32_t s0 = lds_addr(ring);
    auto along_x = [&](int x) { return s0 + (uint32_t)(2 * lk * 64 + (x ^ (16 * lk))) * 8u; };
    auto along_k = [&](int x) { return s0 + wg_at(x); };
    const FarAddr f = {along_x(rx), along_x(rx + 16), along_k(rx), along_k(rx + 16),
                       along_k(cx) + FAR_OPND * 8u, along_k(cx + 16) + FAR_OPND * 8u};
    // the stages are issued in order: the term being issued and its next k
    int q = q0, k = 0, K = 0, ta = 0, left = 0;   // left: stages issued, not yet consumed
    unsigned forms = 0, odd = 0;   // bit i: of the i-th of those, ta; whether it goes to acc1 (NW = 8: to nobody)
    int wr = 0, rd = 0;            // LDS stage of the next issue, of the next products
    constexpr int STEP = NW == 8 ? 32 : 16;
    const double *pa, *pb;         // the term's operands at k
    int da;                        // doubles from one k to the next in Sigma
    uint32_t oa[2], ob[2];
    auto open = [&]() {
        const FarSeg g = seg(q);
        pa = uniform_ptr(g.a);
        pb = uniform_ptr(g.b);
        K = g.K;
        ta = g.ta;
        da = g.ta ? 1 : g.lda;
        far_lanes(g.lda, !g.ta, g.av, v, oa);
        far_lanes(g.ldb, 0, 64, v, ob);
        k = 0;
    };
    open();
    auto issue = [&]() {
        if (q >= q1) return;
        double* st = ring + wr * FAR_STAGE;
        // a half without k of its own repeats the other's loads (the waits
        // count them) and drops them
        const int ks = NW == 8 && half && k + 16 < K ? 16 : 0;
        far_fetch<1>(pa + ks * da, oa, v, st);
        far_fetch<0>(pb + ks, ob, v, st + FAR_OPND);
        forms |= (unsigned)ta << left;
        odd |= (NW == 8 ? (unsigned)(half && ks == 0) : (unsigned)(k >> 4) & 1) << left;
        ++left;
        wr = (wr + 1) & (FAR_STAGES - 1);
        k += STEP;
        pa += STEP * da;
        pb += STEP;
        if (k >= K && ++q < q1) open();
    };
#pragma unroll
    for (int i = 0; i < FAR_STAGES - 1; ++i) issue();
    while (left > 0) {
        far_landed(left - 1);
        asm volatile("s_barrier" ::: "memory");   // ... for every wavefront, and the stage before has been read
        const int t = forms & 1, o = odd & 1;
        forms >>= 1;
        odd >>= 1;
        --left;
        const uint32_t so = (uint32_t)rd * (FAR_STAGE * 8u);
        rd = (rd + 1) & (FAR_STAGES - 1);
        if (!o) far_mma(acc0, f, t, so, issue);
        else if (NW != 8) far_mma(acc1, f, t, so, issue);
        else issue();
    }
}

// Row block rb of a column's FAR tasks: the arrow, then row tiles J+s .. J+2.
__device__ inline void p2_far_row(const Lay& L, int64_t J, int rb, int& d, int& rbl) {
    const int nb64 = L.b / 64, nab = arrow_blocks(L.ap);
    if (rb < nab) { d = ARW; rbl = rb; }
    else { d = L.s(J) - (rb - nab) / nb64; rbl = (rb - nab) % nb64; }
}

template <int NW>
__device__ __forceinline__ bool p2_far(const P2& p, const Sched& sc, int64_t J, int u, double* smem, int* sh, int t) {
    const Lay& L = p.L;
    const int nb64 = L.b / 64, s = p.sw(J);
    const int rb = u / nb64, cb = u % nb64;
    int d, rbl;
    p2_far_row(L, J, rb, d, rbl);
    const int karw = L.ap > 0 ? 1 : 0, n = s + karw;
    auto term = [&](int q) { return q < karw ? ARW : s - (q - karw); };   // q -> tile offset of k
    dbl4 acc[2][2], acc1[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = acc1[i][j] = dbl4{0.0, 0.0, 0.0, 0.0};
    for (int q = 0; q < n;) {
        const int m = p2_ready(sc, n - q, 1, sh, [&](int e, const int*& f, int& t) { p2_sigma_dep(p, J, d, term(q + e), f, t); }, []() {});
        if (m == 0) return false;
        if (q == 0) TRACE(t, 1, wall_clock64());
        if (q + m == n) TRACE(t, 5, wall_clock64());
        far_sum<NW>(acc, acc1, q, q + m, smem, [&](int i) {
            const int e = __builtin_amdgcn_readfirstlane(term(i));
            FarSeg g;
            int64_t lda;
            p2_sigma_rows(L, p.S, J, d, rbl, 64, e, g.a, lda, g.ta, g.av);
            g.lda = (int)lda;
            if (e != ARW) { g.b = p.W + p.wband(J, e) + (int64_t)cb * 64 * L.b; g.ldb = L.b; g.K = e == p.btw ? p.klast : L.b; }
            else { g.b = p.W + p.war(J) + (int64_t)cb * 64 * L.ap; g.ldb = L.ap; g.K = L.ap; }
            return g;
        });
        q += m;
    }
    TRACE(t, 6, wall_clock64());
    double* O;
    int ldo, mv = 64;
    if (d != ARW) { O = p.S + L.band(J, d) + rbl * 64 + (int64_t)cb * 64 * L.b; ldo = L.b; }
    else { O = p.S + L.arrow(J) + rbl * 64 + (int64_t)cb * 64 * L.ap; ldo = L.ap; mv = imin_(64, L.ap - rbl * 64); }
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), v = w & 3;
    const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
    double* o = (double*)uniform_ptr(O);
    auto put = [&](int i, int j, int r, double x) {
        st_coh_s(o, (uint32_t)(32 * (v & 1) + 16 * i + li + (32 * (v >> 1) + 16 * j + 4 * r + lk) * ldo), x);
    };
    // (mv is a multiple of 16)
    if (NW == 8) {
        // each half of the workgroup hands the other one of the two row tiles
        // (i = 1 - half) and stores the other
        const int half = w >> 2;
        double* give = smem + (v * 2 + half) * (8 * 64);
        double* take = smem + (v * 2 + 1 - half) * (8 * 64);
        __syncthreads();   // the last stage has been read
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) give[(4 * j + r) * 64 + l] = half ? acc[0][j][r] : acc[1][j][r];
        __syncthreads();
        if (32 * (v & 1) + 16 * half < mv)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    put(half, j, r, 0.0 - ((half ? acc[1][j][r] : acc[0][j][r]) + take[(4 * j + r) * 64 + l]));
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (32 * (v & 1) + 16 * i < mv)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) put(i, j, r, 0.0 - (acc[i][j][r] + acc1[i][j][r]));
    }
    return true;
}

// ---------------------------------------------------------------------------
// ROW and DIAG
// ---------------------------------------------------------------------------
// The sum in two parts: what is ready first, then the rest.
template <int NW>
__device__ __forceinline__ bool p2_near(const P2& p, const Sched& sc, int kind, int64_t J, int u, double* smem, double* red,
                                        int* sh, int t) {
    const Lay& L = p.L;
    const int C32 = L.b / 32, s = p.sw(J), karw = L.ap > 0 ? 1 : 0;
    const bool row = kind == P2_ROW;
    int rb, cb;
    if (row) { rb = u / C32; cb = u % C32; }
    else tri_decode(u, rb, cb);
    double* O = p.S + L.band(J, row ? 1 : 0) + rb * 32 + (int64_t)cb * 32 * L.b;
    const bool diag = !row && rb == cb;
    // Sigma_JJ starts as X^T X (Phase 1): read now, its round trip behind the waits
    constexpr int NTH = P2Cfg<NW>::NTH;
    double ov[1024 / NTH];
#pragma unroll
    for (int q = 0; q < 1024 / NTH; ++q) {
        const int e = threadIdx.x + NTH * q;
        ov[q] = row ? 0.0 : ld_coh(O + (e & 31) + (int64_t)(e >> 5) * L.b);
    }
    dbl4 acc[2][2], acc1[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = acc1[i][j] = dbl4{0.0, 0.0, 0.0, 0.0};
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double* sw = smem + w * WG_WAVE;
    // term e (a band tile offset or ARW) of the sum.  Both operands run along
    // k: row tile J+1 of Sigma is column J+1 transposed (its diagonal tile is
    // symmetric and full), and in DIAG Sigma's columns stand for the rows of
    // the (symmetric) result.
    auto term = [&](int e) {
        const int ld = e == ARW ? L.ap : L.b;
        Seg g;
        g.a = p.S + (e == ARW ? L.arrow(row ? J + 1 : J) : L.band(row ? J + 1 : J, row ? e - 1 : e)) + (int64_t)rb * 32 * ld;
        g.b = p.W + (e == ARW ? p.war(J) : p.wband(J, e)) + (int64_t)cb * 32 * ld;
        g.lda = g.ldb = ld;
        g.K = e == ARW ? L.ap : e == p.btw ? p.klast : L.b;
        return g;
    };
    // the counter of its Sigma operand
    auto dep = [&](int e, const int*& f, int& t) {
        if (row) { p2_sigma_dep(p, J, 1, e, f, t); return; }
        f = p2_counter(p, J, e);
        t = p2_target(L, e);
    };
    // two parts: ROW the tiles from J+2 on and the arrow, then J+1; DIAG the
    // arrow and the tiles from J+3 on, then J+2 and J+1, as FAR(J) ends on row
    // tile J+2 - but with fewer than three band tiles below, FAR(J) is early and
    // J+2 belongs to part one (nb 6,000, w 256, tile 128: 564 against 601 us;
    // w 553 1.92 against 1.98 ms the other way)
    const int e2 = imin_(s, !row && s >= 3 ? 2 : 1);   // part two: tile offsets e2 .. 1
    const int n1 = s - e2 + karw;
    auto off1 = [&](int q) { return q < karw ? ARW : s - (q - karw); };
    auto len = [&](int e) { return e == p.btw ? p.klast : L.b; };
    if (n1 > 0) {
        const int klen = L.ap + (s > e2 ? (s - e2 - 1) * L.b + len(s) : 0);
        if (!wave_sum<NW>(acc, acc1, n1, klen, sw, [&](int q) { return term(off1(q)); }, [&](auto&& pre) {
                return p2_all_ready(sc, n1, sh, [&](int q, const int*& f, int& t) { dep(off1(q), f, t); }, pre);
            }))
            return false;
    }
    if (e2 > 0) {
        if (!wave_sum<NW>(acc, acc1, e2, len(1) + (e2 > 1 ? len(2) : 0), sw, [&](int q) { return term(e2 - q); }, [&](auto&& pre) {
                return p2_all_ready(sc, e2, sh, [&](int q, const int*& f, int& t) { dep(e2 - q, f, t); }, pre);
            }))
            return false;
    }
    if (NW != 8)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] += acc1[i][j];
    wave_reduce<NW>(acc, smem, red);
    TRACE(t, 6, wall_clock64());
#pragma unroll
    for (int q = 0; q < 1024 / NTH; ++q) {
        const int e = threadIdx.x + NTH * q, i = e & 31, j = e >> 5;
        if (diag && i < j) continue;
        red[j * WR_LD + i] = ov[q] - red[j * WR_LD + i];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 1024; e += NTH) {
        const int i = e & 31, j = e >> 5;
        const double v = diag && i < j ? red[i * WR_LD + j] : red[j * WR_LD + i];
        st_coh(O + i + (int64_t)j * L.b, v);
        if (!row && !diag) {   // mirrored, down its columns
            const int i2 = e & 31, j2 = e >> 5;
            st_coh(p.S + L.band(J, 0) + (cb * 32 + i2) + (int64_t)(rb * 32 + j2) * L.b, red[i2 * WR_LD + j2]);
        }
    }
    return true;
}

// Takes tickets until there are none (true) or the kernel must stop.
template <int NW>
__device__ inline bool p2_run(const P2& p, const Sched& sc, double* smem, int* sh) {
    double* red = smem + P2Cfg<NW>::STAGE;
    const Lay& L = p.L;
    const int64_t N = L.nt;
    for (;;) {
        const int t = sched_next(sc, p.ntasks, &sh[0]);
        if (t < 0) return true;   // (or an error, which every later wait meets)
        TRACE(t, 0, wall_clock64());
        int64_t q;
        int base;
        if (t >= p.off_q0) {
            q = p.q0 + (t - p.off_q0) / p.g_tasks;
            if (q > N - 1 - p.jf) q = N - 1 - p.jf;
            base = p.off_q0 + (int)(q - p.q0) * p.g_tasks;
        } else {
            // p2_base is a q^2 + b q + c from q = 1 on: its root, set right
            // for the rounding
            const double nb64 = L.b / 64, nn = 0.5 * nb64 * nb64, bb = (double)p2_base(L, 2) - (double)p2_base(L, 1) - 3.0 * nn;
            const double cc = (double)p2_base(L, 1) - nn - bb;
            q = (int64_t)((sqrt(fmax(bb * bb + 4.0 * nn * (t - cc), 0.0)) - bb) / (2.0 * nn));
            q = q < 0 ? 0 : q > p.q0 - 1 ? p.q0 - 1 : q;
            while (q > 0 && p2_base(L, q) > t) --q;
            while (q < p.q0 - 1 && p2_base(L, q + 1) <= t) ++q;
            base = (int)p2_base(L, q);
        }
        const int64_t G = N - 1 - q;
        int u = t - base;
        // the group's parts in turn: [FAR(N-1)], FAR(G-1) but for row tile
        // G+1, ROW(G), the rest of FAR(G-1), DIAG(G)
        int64_t J = G;
        int d = 0, kind = P2_DIAG;
        const int n0 = G == N - 1 ? p2_far_tasks(L, G) : 0;
        const int n1 = G > p.jf ? p2_far_tasks(L, G - 1) : 0, n2 = G > p.jf ? p2_far2_tasks(L, G - 1) : 0, nr = p2_row_tasks(L, G);
        if (u < n0) {
            kind = P2_FAR;
        } else if ((u -= n0) < n1 - n2) {
            kind = P2_FAR;
            J = G - 1;
        } else if ((u -= n1 - n2) < nr) {
            kind = P2_ROW;
            d = 1;
        } else if ((u -= nr) < n2) {
            kind = P2_FAR;
            J = G - 1;
            u += n1 - n2;
        } else {
            u -= n2;
        }
        bool ok;
        if (kind == P2_FAR) {
            int rbl;
            p2_far_row(L, J, u / (L.b / 64), d, rbl);
            if (d == ARW) d = p2_arw(L);
            ok = p2_far<NW>(p, sc, J, u, smem, &sh[1], t);
        } else {
            ok = p2_near<NW>(p, sc, kind, J, u, smem, red, &sh[1], t);
        }
        if (!ok) return false;
        sched_signal(sc, p.cnt + J * p2_ctr(L) + d, t);
        TRACE(t, 2, wall_clock64());
        TRACE(t, 3, (unsigned long long)kind | ((unsigned long long)J << 8) | ((unsigned long long)blockIdx.x << 40));
        TRACE(t, 7, (unsigned long long)__smid());
    }
}
