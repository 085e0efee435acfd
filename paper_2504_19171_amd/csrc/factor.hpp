// The factor of the band and arrow as one persistent launch over 64 x 64
// blocks.
//
// The matrix is cut into chunks of 64 columns, whatever the tile size (tiles
// are multiples of 64).  Block (i, c) is rows 64 i.., columns 64 c.. of the
// band (i - c <= Wc = ceil(w / 64): the blocks below that hold only entries
// outside the element band, which stay zero), or rows 64 r.. of the arrow.
//
// What bounds the factor is the chain of diagonal blocks, one after the
// other, so one workgroup per matrix (the chain) does nothing else: per chunk
// it factors the 64 x 64 diagonal block, solves the block row below it and
// applies that row to the next diagonal block, all in registers and LDS, with
// no hand-off through memory on the way (fac_chain).  Every other block is
// left-looking: a task reads the block once, subtracts the products of the
// finished blocks to its left, solves against the chunk's diagonal block and
// writes it once (fac_task).  The two meet two block rows below the diagonal:
//   G(i, c), i >= c + 3, and every arrow block: the whole sum over k < c, then
//     the solve with chunk c;
//   P(i, j), j in {i - 2, i - 1, i}: the early part of the sum of the blocks
//     that are due soonest, written back in place;
//   H1(i): the rest of block (i, i - 2) and its solve (not stored), then its
//     product into the diagonal block (i, i), which the chain takes over;
//   H0(i): the same solve again, stored once H1(i) has read what it replaces,
//     and its product into block (i, i - 1), which the chain takes over too.
//     The two run side by side, because either alone would be late for the
//     chain;
//   C(r, s; q): chunks 4q .. 4q + 3 into corner block (r, s).
// Tasks are dealt by tickets in the order of fac_group; a task waits only for
// tasks of smaller tickets and for the chain, the chain only for tasks, which
// have larger tickets than it: it gets no further unless a second workgroup of
// the launch runs.  A launch has at least two per matrix when it has tasks, next
// to each other, so of all launches that run at once those that cannot go on
// hold one workgroup of the chip each; with fewer launches than workgroups fit
// it (256 and more) the others end and make room.  Such a wait counts towards
// the spin limit.
// Without blocks below the diagonal ones (w = 0, or a single chunk) the chunks
// do not depend on each other: each is a chain of its own, and these take the
// first tickets (nb 200,000, w 0, tile 64: 16.9 ms with one chain for all, 0.15
// ms so).
//
// Every block is written once in its final form (P and H parts before that
// are read only by the task or chain that goes on with them) with
// device-coherent stores, and read by others only after its flag is up, with
// device-coherent loads (see persist.hpp).
#pragma once
#include "common.hpp"
#include "persist.hpp"
#include "factor16.hpp"

#define FC 64          // chunk width
#define FAC_NT 256     // threads per workgroup (4 wavefronts)
#define FAC_STAGES 4   // 16-column operand stages in LDS

struct FacCtx {
    double* Lm;
    Lay L;
    int c64;    // chunks per tile (1 .. 4)
    uint32_t dm, ds;   // c / c64 = (c * dm) >> ds: a division would cost hundreds of cycles on the chain
    int nc;     // chunks that hold real columns
    int wc;     // block half-bandwidth
    int w1;     // max(wc, 1): row length of fl
    int na;     // arrow row blocks
    int col0;   // first column's number in the matrix
    double* Yd; // Y_p of every chunk, 4 x 256 doubles in operand order
    int* po;    // [nc * 4]   row tile t of chunk c's diagonal block and Y_t are in memory
    int* fl;    // [nc * w1]  block (i, k) final at fl[i * w1 + i - k - 1]: 4
    int* fa;    // [na * nc]  arrow block (r, k) final: 4
    int* hx;    // [nc * 2]   H0(i), H1(i) done
    int* pp;    // [nc * 4]   P(i, i), P(i, i - 1), P(i, i - 2) done; H1(i) has read block (i, i - 2)
    int* cc;    // [na (na + 1) / 2]  groups of four chunks in a corner block
};
__host__ __device__ inline int fac_chunks(const Lay& L) { return (int)((L.nb + FC - 1) / FC); }
__host__ __device__ inline int fac_wc(const Lay& L) {
    const int64_t wc = (L.w + FC - 1) / FC, m = fac_chunks(L) - 1;
    return (int)(wc < m ? wc : m);
}
// Flag ints of one factorization (from po on, contiguous).
__host__ __device__ inline int64_t fac_ints(const Lay& L) {
    const int64_t nc = fac_chunks(L), wc = fac_wc(L), na = arrow_blocks(L.ap);
    return nc * 4 + nc * (wc > 1 ? wc : 1) + na * nc + nc * 2 + nc * 4 + na * (na + 1) / 2;
}
__host__ __device__ inline FacCtx fac_ctx(const Lay& L, double* Lm, double* Yd, int* flags) {
    FacCtx x;
    x.Lm = Lm;
    x.L = L;
    x.c64 = L.b / FC;
    x.dm = x.c64 == 3 ? 0xAAAAAAABu : 1u;
    x.ds = x.c64 == 3 ? 33 : (x.c64 == 4 ? 2 : x.c64 - 1);
    x.nc = fac_chunks(L);
    x.wc = fac_wc(L);
    x.w1 = x.wc > 1 ? x.wc : 1;
    x.na = arrow_blocks(L.ap);
    x.col0 = 0;
    x.Yd = Yd;
    x.po = flags;
    x.fl = x.po + x.nc * (int64_t)4;
    x.fa = x.fl + x.nc * (int64_t)x.w1;
    x.hx = x.fa + x.na * (int64_t)x.nc;
    x.pp = x.hx + x.nc * (int64_t)2;
    x.cc = x.pp + x.nc * (int64_t)4;
    return x;
}

// Tasks of group c (see fac_pick for their order): the tasks that end with
// the solve of chunk c, and the early sums that end with its blocks.
__host__ __device__ inline int fac_group(const FacCtx& x, int c) {
    const int left = imin_(x.wc, x.nc - 1 - c);   // block rows below the diagonal
    int n = x.na;
    if (left >= 2) n += 2;                        // H0, H1 (c + 2)
    if (left >= 3) n += left - 2 + 2;             // G(c + 3 ..), P(c + 3, c + 2), P(c + 3, c + 3)
    if (left >= 4) n += 1;                        // P(c + 4, c + 2)
    if ((c & 3) == 3 || c == x.nc - 1) n += x.na * (x.na + 1) / 2;
    return n;
}
// Leading chunks whose groups are all alike (but for the corner tasks of
// every fourth), rounded down to a multiple of four.
__host__ __device__ inline int fac_full4(const FacCtx& x) { return imax_(0, x.nc - 1 - imax_(x.wc, 4)) & ~3; }
// Chains: tickets in front of the tasks.
__host__ __device__ inline int fac_chains(const FacCtx& x) { return x.wc == 0 ? x.nc : 1; }
__host__ __device__ inline int64_t fac_tasks(const FacCtx& x) {
    const int f4 = fac_full4(x);
    int64_t t = 0;
    if (f4 > 0)
        for (int c = 0; c < 4; ++c) t += fac_group(x, c);
    t *= f4 / 4;
    for (int c = f4; c < x.nc; ++c) t += fac_group(x, c);
    return t;
}

// ---------------------------------------------------------------------------
// LDS
// ---------------------------------------------------------------------------
struct ChainSmem {
    double Y[2][4][16 * 17];   // Y_p of the chunk (by its parity), element (i, j) at j * 17 + i
    double Lt[2][6][256];      // tile (t, p), t > p, of the diagonal block in operand order (r * 64 + lane)
    double R[4][4][256];       // strip s, panel p of the block row below, in operand order
    double X[2][256];          // what tiles (3, 1) and (3, 2) of the diagonal block lose to R
    int w[32];                 // progress words (CW_*)
};
enum {
    CW_Y = 0,     // [4] chunks whose Y_p is there
    CW_L = 4,     // [4] 4 c + panels of row t there
    CW_R = 8,     // [4] 4 c + panels of strip s there
    CW_D = 12,    // [4] chunks for which wavefront t has read R
    CW_X = 16     // [1] chunks whose X is there
};
struct TaskSmem {
    double st[FAC_STAGES][2][16 * 64];   // per stage: 16 columns of the column-side rows, then of the row-side rows
};
struct FacSmem {
    union {
        ChainSmem ch;
        TaskSmem tk;
    };
    int sh;     // scheduler broadcast
    int n;      // blocks ready (fac_acc)
    int dead;   // a wait of this workgroup failed
};

// ---------------------------------------------------------------------------
// Addresses
// ---------------------------------------------------------------------------
// Tile of chunk c.
__device__ inline int fac_tile(const FacCtx& x, int c) { return (int)(((uint64_t)(uint32_t)c * x.dm) >> x.ds); }
// Block (i, c) of the band, leading dimension b.
__device__ inline double* fac_band(const FacCtx& x, int i, int c) {
    const int I = fac_tile(x, i), J = fac_tile(x, c);
    return x.Lm + x.L.band(J, I - J) + (i - I * x.c64) * FC + (int64_t)(c - J * x.c64) * FC * x.L.b;
}
// Arrow block (r, c), leading dimension a_p.
__device__ inline double* fac_arrow(const FacCtx& x, int r, int c) {
    const int J = fac_tile(x, c);
    return x.Lm + x.L.arrow(J) + r * FC + (int64_t)(c - J * x.c64) * FC * x.L.ap;
}
// A block row: band row i, or arrow row block r.
struct FacRow {
    int i;   // band row, or -1 - r
};
__device__ inline const double* fac_ptr(const FacCtx& x, FacRow w, int k) {
    return w.i >= 0 ? fac_band(x, w.i, k) : fac_arrow(x, -1 - w.i, k);
}
__device__ inline int fac_ld(const FacCtx& x, FacRow w) { return w.i >= 0 ? x.L.b : x.L.ap; }
__device__ inline int fac_valid(const FacCtx& x, FacRow w) {
    return w.i >= 0 ? FC : imin_(FC, x.L.ap - FC * (-1 - w.i));
}
__device__ inline int* fac_flag(const FacCtx& x, FacRow w, int k) {
    return w.i >= 0 ? x.fl + (int64_t)w.i * x.w1 + (w.i - k - 1) : x.fa + (int64_t)(-1 - w.i) * x.nc + k;
}

// Words in LDS that other wavefronts write: volatile, and through the LDS
// address space (a volatile access through a generic pointer stays a FLAT
// instruction, which waits for every memory access in flight).
typedef volatile __attribute__((address_space(3))) int lds_word_t;
__device__ inline int fac_lds_get(const int* p) { return *(lds_word_t*)p; }
__device__ inline void fac_lds_set(int* p, int v) { *(lds_word_t*)p = v; }

__device__ inline void fac_bar() { asm volatile("s_barrier" ::: "memory"); }
__device__ inline void fac_vm0() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ inline void fac_up(int* f, int v) {
    __hip_atomic_store((GLOBAL_AS int*)f, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One wavefront waits until *f >= target; false when the kernel must stop.
__device__ inline bool fac_wait1(const Sched& sc, const int* f, int target) {
    int v = __builtin_amdgcn_readfirstlane(ld_coh_i(f));
    if (v >= target) return true;
    const int64_t t0 = wall_clock64();
    for (unsigned n = 0;; ++n) {
        v = __builtin_amdgcn_readfirstlane(ld_coh_i(f));
        if (v >= target) return true;
        if ((n & 15) == 15) {
            if (__builtin_amdgcn_readfirstlane(ld_coh_i(sc.err)) != 0) return false;
            if (wall_clock64() - t0 > sc.spin_limit) {
                set_error_once(sc.err, STILES_ETIMEOUT);
                return false;
            }
        }
        __builtin_amdgcn_s_sleep(1);
    }
}
// Row tiles of chunk c's diagonal block in memory (the leading ones), at least
// `need`; 0: stop.
__device__ inline int fac_panels(const Sched& sc, const int* po, int need) {
    const int lane = threadIdx.x & 63;
    int64_t t0 = -1;
    for (unsigned n = 0;; ++n) {
        const uint64_t m = __ballot(ld_coh_i(po + (lane & 3)) != 0) & 15;
        const int have = __builtin_ctz(~(unsigned)m);
        if (have >= need) return have;
        if (t0 < 0) t0 = wall_clock64();
        if ((n & 15) == 15) {
            if (__builtin_amdgcn_readfirstlane(ld_coh_i(sc.err)) != 0) return 0;
            if (wall_clock64() - t0 > sc.spin_limit) {
                set_error_once(sc.err, STILES_ETIMEOUT);
                return 0;
            }
        }
        __builtin_amdgcn_s_sleep(1);
    }
}
// Every wavefront says whether its waits succeeded; false for all when one failed.
__device__ inline bool fac_agree(FacSmem& sm, bool ok) {
    if (!ok) sm.dead = 1;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    fac_bar();
    return __builtin_amdgcn_readfirstlane(fac_lds_get(&sm.dead)) == 0;
}

// ---------------------------------------------------------------------------
// The sum of products of a task
// ---------------------------------------------------------------------------
// Wavefront v owns rows 16 v .. 16 v + 15 of a 64 x 64 block (its strip), as
// four 16 x 16 tiles: element r of z[t] is (row 16 v + li, column
// 16 t + 4 r + lk), the transposed product on the matrix cores, so that every
// access to memory runs down a column, and so that a solved strip is already
// the operand of the next product.

// The same value, but opaque: offsets formed from it are formed where they are
// used, not hoisted out of the kernel's task loop (where they would only
// occupy registers).
__device__ inline int fac_opaque(int v) {
    v = __builtin_amdgcn_readfirstlane(v);
    asm volatile("" : "+s"(v));
    return v;
}

// This lane, opaque for the same reason.
__device__ inline int fac_lane() {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
    return l;
}

// Bytes a lane takes from memory per load into LDS: 16 where L starts at a
// multiple of 16 bytes, which every block then does (tile sizes, a_p and leading
// dimensions are even), else 4: the caller may place L at any double (nb 100,000
// w 1,024 a 100 tile 256: 19.5 and 24.9 ms with the copy of A; nb 31,987 w 32 4.6
// and 5.2).
#define FAC_WIDE 16
#define FAC_NARROW 4
__host__ __device__ inline bool fac_wide(const void* Lm) { return ((uintptr_t)Lm & 15) == 0; }

// One kilobyte (128 doubles) straight into LDS, double p of it from at(p) (pairs
// p, p + 1, p even, are contiguous): one load of 16 bytes a lane, or four of 4.
template <int LD, class F>
__device__ inline void fac_fetch(int l, double* st, F&& at) {
    if constexpr (LD == FAC_WIDE) {
        __builtin_amdgcn_global_load_lds((const void*)at(2 * l), (lds_void_t*)st, 16, 0, 16);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            __builtin_amdgcn_global_load_lds((const void*)((const char*)at(32 * j + (l >> 1)) + 4 * (l & 1)),
                                             (lds_void_t*)(st + 32 * j), 4, 0, 16);
    }
}

// Issue the loads of stage `q` (16 columns) of block column k: columns 4 v ..
// 4 v + 3 of the column-side rows and of the row-side rows, straight into LDS
// (element (row x, column k) at k * 64 + (x ^ 16 (k & 3)): the four columns
// that one matrix-core operand takes fall in different banks).  Rows past va
// (vb) repeat the last two.
template <int LD>
__device__ inline void fac_issue(const double* A, int lda, int va, const double* B, int ldb, int vb, int q,
                                 double (*st)[16 * 64]) {
    const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = fac_lane();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        auto from = [&](const double* P, int ld, int valid) {
            return [=](int p) {
                const int half = p >> 6, row = (p & 63) ^ (16 * ((2 * u + half) & 3));
                return P + imin_(row & ~1, valid - 2) + (p & 1) + (int64_t)(16 * q + 4 * v + 2 * u + half) * ld;
            };
        };
        fac_fetch<LD>(l, st[0] + (4 * v + 2 * u) * 64, from(A, lda, va));
        fac_fetch<LD>(l, st[1] + (4 * v + 2 * u) * 64, from(B, ldb, vb));
    }
}
template <int LD>
__device__ inline void fac_issue_a(const double* A, int lda, int q, double* st) {
    const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = fac_lane();
#pragma unroll
    for (int u = 0; u < 2; ++u)
        fac_fetch<LD>(l, st + (4 * v + 2 * u) * 64, [=](int p) {
            const int half = p >> 6;
            return A + ((p & 63) ^ (16 * ((2 * u + half) & 3))) + (int64_t)(16 * q + 4 * v + 2 * u + half) * lda;
        });
}

typedef double dbl2 __attribute__((ext_vector_type(2)));
// Operands of eight columns (two matrix-core steps): .x of the first four
// columns, .y of the next four.  Reads and their wait in one block, as the
// compiler would also wait for every load into LDS still in flight.
__device__ inline void fac_read(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t b, dbl2 (&a)[4], dbl2& bv) {
    asm volatile(
        "ds_read2st64_b64 %4, %9 offset1:4\n\t"
        "ds_read2st64_b64 %0, %5 offset1:4\n\t"
        "ds_read2st64_b64 %1, %6 offset1:4\n\t"
        "ds_read2st64_b64 %2, %7 offset1:4\n\t"
        "ds_read2st64_b64 %3, %8 offset1:4\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(bv)
        : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(b)
        : "memory");
}
__device__ inline void fac_read_a(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, dbl2 (&a)[4]) {
    asm volatile(
        "ds_read2st64_b64 %0, %4 offset1:4\n\t"
        "ds_read2st64_b64 %1, %5 offset1:4\n\t"
        "ds_read2st64_b64 %2, %6 offset1:4\n\t"
        "ds_read2st64_b64 %3, %7 offset1:4\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
        : "v"(a0), "v"(a1), "v"(a2), "v"(a3)
        : "memory");
}

// Wait until the oldest of this wavefront's load stages has landed, `later`
// stages (PER loads of 16 bytes a lane each, or four times as many of 4) issued
// after it.
template <int LD, int PER>
__device__ inline void fac_landed(int later) {
    constexpr int N = PER * (FAC_WIDE / LD);   // 2 to 16; the counter goes to 63
    if (later >= 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * N) : "memory");
    else if (later == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * N) : "memory");
    else if (later == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// acc[t] += (row w, k) (col-side row u, k)^T over k0 <= k < k1, tiles t < nt,
// as the blocks' flags come up.  act: this wavefront's strip has rows.
template <int LD>
__device__ inline bool fac_acc(const FacCtx& x, const Sched& sc, FacSmem& sm, dbl4 (&acc)[4], FacRow w, FacRow u,
                               int k0, int k1, int nt, bool act) {
    const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = fac_lane(), li = lane & 15, lk = lane >> 4;
    const int ldw = fac_ld(x, w), ldu = fac_ld(x, u), vw = fac_valid(x, w), vu = fac_valid(x, u);
    uint32_t oa[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) oa[t] = lds_addr(sm.tk.st[0][0]) + 8u * (uint32_t)(lk * 64 + 16 * (t ^ lk) + li);
    const uint32_t ob = lds_addr(sm.tk.st[0][1]) + 8u * (uint32_t)(lk * 64 + 16 * (v ^ lk) + li);
    if (LD == FAC_NARROW) fac_vm0();   // (with the block's own loads there would be more in flight than can be counted)
    for (int k = k0; k < k1;) {
        // leading blocks that are ready, up to 32: lanes 0..31 read the row
        // side's flags, lanes 32..63 the column side's
        if (v == 0) {
            const int m = imin_(k1 - k, 32), e = imin_(lane & 31, m - 1);
            const int* f = lane < 32 ? fac_flag(x, w, k + e) : fac_flag(x, u, k + e);
            int n = 0;
            int64_t t0 = -1;
            for (unsigned polls = 0;; ++polls) {
                const uint64_t b = __ballot(ld_coh_i(f) >= 4);
                const uint32_t both = (uint32_t)b & (uint32_t)(b >> 32);
                n = both == 0xffffffffu ? 32 : __builtin_ctz(~both);
                n = imin_(n, m);
                if (n > 0) break;
                if (t0 < 0) t0 = wall_clock64();
                if ((polls & 15) == 15) {
                    if (__builtin_amdgcn_readfirstlane(ld_coh_i(sc.err)) != 0) break;
                    if (wall_clock64() - t0 > sc.spin_limit) {
                        set_error_once(sc.err, STILES_ETIMEOUT);
                        break;
                    }
                }
                __builtin_amdgcn_s_sleep(1);
            }
            if (lane == 0) sm.n = n;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        fac_bar();
        const int n = __builtin_amdgcn_readfirstlane(fac_lds_get(&sm.n));
        if (n == 0) return false;
        const int total = 4 * n;
        auto issue = [&](int it) {
            const int kk = k + (it >> 2);
            fac_issue<LD>(uniform_ptr(fac_ptr(x, u, kk)), ldu, vu, uniform_ptr(fac_ptr(x, w, kk)), ldw, vw, it & 3,
                      sm.tk.st[it & 3]);
        };
#pragma unroll
        for (int it = 0; it < FAC_STAGES - 1; ++it) issue(it);   // a block has four stages
        for (int it = 0; it < total; ++it) {
            fac_landed<LD, 4>(imin_(total - 1 - it, FAC_STAGES - 2));
            fac_bar();   // ... for every wavefront, and stage it - 1 has been read
            if (it + FAC_STAGES - 1 < total) issue(it + FAC_STAGES - 1);
            if (act) {
                const uint32_t so = (uint32_t)(it & 3) * (uint32_t)(2 * 16 * 64 * 8);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    dbl2 a[4], b;
                    const uint32_t o = so + (uint32_t)h * (8 * 64 * 8);
                    fac_read(oa[0] + o, oa[1] + o, oa[2] + o, oa[3] + o, ob + o, a, b);
                    if (nt == 4) {
#pragma unroll
                        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].x, b.x, acc[t], 0, 0, 0);
#pragma unroll
                        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].y, b.y, acc[t], 0, 0, 0);
                    } else {
#pragma unroll
                        for (int t = 0; t < 3; ++t)
                            if (t < nt) {
                                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].x, b.x, acc[t], 0, 0, 0);
                                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].y, b.y, acc[t], 0, 0, 0);
                            }
                    }
                }
            }
        }
        k += n;
    }
    fac_bar();   // every wavefront has read the last stage: the LDS may be reused
    return true;
}

// Strip rows of a block at `base` (leading dimension ld), tiles t < nt.
__device__ inline void fac_load(const double* base, int ld, int v, dbl4 (&z)[4], int nt) {
    ld = fac_opaque(ld);
    const int lane = fac_lane(), li = lane & 15, lk = lane >> 4;
    const double* b = uniform_ptr(base);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (t < nt) {
#pragma unroll
            for (int r = 0; r < 4; ++r) z[t][r] = ld_coh_s(b, (uint32_t)((16 * v + li) + (16 * t + 4 * r + lk) * ld));
        }
}
__device__ inline void fac_store(double* base, int ld, int v, const dbl4 (&z)[4], int nt) {
    ld = fac_opaque(ld);
    const int lane = fac_lane(), li = lane & 15, lk = lane >> 4;
    double* b = (double*)uniform_ptr(base);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (t < nt) {
#pragma unroll
            for (int r = 0; r < 4; ++r) st_coh_s(b, (uint32_t)((16 * v + li) + (16 * t + 4 * r + lk) * ld), z[t][r]);
        }
}

// Solve of a strip with the diagonal block of chunk c, row tile by row tile as
// the chain announces them: Z_t^T -= sum_{p < t} L_tp R_p^T, o[t] = R_t^T =
// Y_t Z_t^T.  The strip never leaves the wavefront's registers.
__device__ inline bool fac_solve(const FacCtx& x, const Sched& sc, int c, dbl4 (&z)[4], dbl4 (&o)[4]) {
    const int lane = fac_lane(), li = lane & 15, lk = lane >> 4;
    const double* D = uniform_ptr(fac_band(x, c, c));
    const double* Y = uniform_ptr(x.Yd + (int64_t)c * 1024);
    const int b = fac_opaque(x.L.b);
    double yv[4][4], lv[4][4][4];
    auto fetch = [&](int t) {
#pragma unroll
        for (int p = 0; p < t; ++p)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                lv[t][p][r] = ld_coh_s(D, (uint32_t)((16 * t + li) + (16 * p + 4 * r + lk) * b));
#pragma unroll
        for (int r = 0; r < 4; ++r) yv[t][r] = ld_coh_s(Y, (uint32_t)(t * 256 + r * 64 + lane));
    };
    auto step = [&](int t) {
        dbl4 q = dbl4{0.0, 0.0, 0.0, 0.0}, e = q;   // two chains each
#pragma unroll
        for (int p = 0; p < t; ++p) {
            z[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-lv[t][p][0], o[p][0], z[t], 0, 0, 0);
            q = __builtin_amdgcn_mfma_f64_16x16x4f64(-lv[t][p][1], o[p][1], q, 0, 0, 0);
            z[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-lv[t][p][2], o[p][2], z[t], 0, 0, 0);
            q = __builtin_amdgcn_mfma_f64_16x16x4f64(-lv[t][p][3], o[p][3], q, 0, 0, 0);
        }
        if (t > 0) z[t] += q;
        q = dbl4{0.0, 0.0, 0.0, 0.0};
        e = __builtin_amdgcn_mfma_f64_16x16x4f64(yv[t][0], z[t][0], e, 0, 0, 0);
        q = __builtin_amdgcn_mfma_f64_16x16x4f64(yv[t][1], z[t][1], q, 0, 0, 0);
        e = __builtin_amdgcn_mfma_f64_16x16x4f64(yv[t][2], z[t][2], e, 0, 0, 0);
        q = __builtin_amdgcn_mfma_f64_16x16x4f64(yv[t][3], z[t][3], q, 0, 0, 0);
        o[t] = e + q;
    };
    const int* po = x.po + (int64_t)c * 4;
    int have = fac_panels(sc, po, 1);
    if (have == 0) return false;
    fetch(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        // the next tile's operands on their way while this one is solved, if they are there
        const bool ahead = have > t + 1;
        if (t < 3 && ahead) fetch(t + 1);
        step(t);
        if (t < 3 && !ahead) {
            have = fac_panels(sc, po, t + 2);
            if (have == 0) return false;
            fetch(t + 1);
        }
    }
    return true;
}

// Which task is index u of group c.
enum { FT_G = 0, FT_H0, FT_H1, FT_P, FT_ARROW, FT_CORNER };
struct FacTask {
    int kind, i, j;   // G: block (i, c); P: block (i, j); ARROW: row block i; CORNER: block (i, j)
};
__device__ inline FacTask fac_pick(const FacCtx& x, int c, int u) {
    const int left = imin_(x.wc, x.nc - 1 - c);
    FacTask k;
    k.i = c + 2;
    k.j = c;
    if (left >= 2) {
        if (u < 2) { k.kind = u == 0 ? FT_H1 : FT_H0; return k; }
        u -= 2;
    }
    if (left >= 3) {
        k.i = c + 3;
        if (u == 0) { k.kind = FT_G; return k; }
        k.kind = FT_P;
        if (u < 3) { k.j = c + 1 + u; return k; }
        u -= 3;
    }
    if (left >= 4) {
        k.i = c + 4;
        if (u == 0) { k.kind = FT_G; return k; }
        k.kind = FT_P;
        if (u == 1) { k.j = c + 2; return k; }
        u -= 2;
        if (u < left - 4) { k.kind = FT_G; k.i = c + 5 + u; return k; }
        u -= left - 4;
    }
    if (u < x.na) { k.kind = FT_ARROW; k.i = u; return k; }
    k.kind = FT_CORNER;
    tri_decode(u - x.na, k.i, k.j);
    return k;
}

// Task u of group c; false when the kernel must stop.  ticket: the launch's
// ticket (the test hook Sched::withhold names one whose signal is not sent).
// The kinds share one copy of the sum and of the solve: with a copy for each,
// the kernel's code would not fit the instruction cache.
template <int LD>
__device__ inline bool fac_task(const FacCtx& x, const Sched& sc, FacSmem& sm, int c, int u, int ticket) {
    const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const FacTask k = fac_pick(x, c, u);
    const int b = x.L.b, ap = x.L.ap;
    const bool quiet = ticket == sc.withhold;
    const bool hand = k.kind == FT_H0 || k.kind == FT_H1;
    const int i = k.i;
    // rows of the block, rows of its columns, the range of k, tiles per strip
    FacRow w{i}, cr{c};
    int k0, k1 = c, nt = 4, ld = b;
    double* O;
    if (k.kind == FT_G) {
        k0 = i - x.wc;
        O = fac_band(x, i, c);
    } else if (k.kind == FT_ARROW) {
        w.i = -1 - i;
        k0 = c - x.wc;
        O = fac_arrow(x, i, c);
        ld = ap;
    } else if (k.kind == FT_P) {
        cr.i = k.j;
        k0 = i - x.wc;
        k1 = c + 1;
        nt = i == k.j ? v + 1 : 4;
        O = fac_band(x, i, k.j);
    } else if (k.kind == FT_CORNER) {
        w.i = -1 - i;
        cr.i = -1 - k.j;
        k0 = c & ~3;
        k1 = c + 1;
        const int n = fac_valid(x, cr) / 16;
        nt = i == k.j ? imin_(v + 1, n) : n;
        O = x.Lm + x.L.corner() + FC * i + (int64_t)FC * k.j * ap;
        ld = ap;
    } else {   // block (i, i - 2): what P(i, i - 2) left
        k0 = x.wc >= 3 ? i - 3 : c;
        O = fac_band(x, i, c);
        if (x.wc >= 4 && i >= 4 && !sched_wait(sc, x.pp + i * (int64_t)4 + 2, 1, &sm.sh)) return false;
    }
    k0 = imax_(k0, 0);
    const bool act = 16 * v < fac_valid(x, w);   // this wavefront's strip has rows
    dbl4 acc[4], z[4], o[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = z[t] = dbl4{0.0, 0.0, 0.0, 0.0};
    if (act && k.kind != FT_CORNER) fac_load(O, ld, v, z, nt);
    if (k.kind == FT_H1) {   // H0 may replace the block from now on
        fac_vm0();
        fac_bar();
        if (threadIdx.x == 0) fac_up(x.pp + i * (int64_t)4 + 3, 1);
    }
    if (!fac_acc<LD>(x, sc, sm, acc, w, cr, k0, k1, nt, act)) return false;
    int* cnt = x.cc + (i * (i + 1) / 2 + k.j);
    if (k.kind == FT_CORNER) {
        if (!sched_wait(sc, cnt, c >> 2, &sm.sh)) return false;
        if (act) fac_load(O, ld, v, z, nt);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) z[t] -= acc[t];
    if (k.kind == FT_P || k.kind == FT_CORNER) {
        if (act) fac_store(O, ld, v, z, nt);
        fac_vm0();
        fac_bar();
        if (threadIdx.x == 0 && !quiet) {
            if (k.kind == FT_P) fac_up(x.pp + i * (int64_t)4 + (i - k.j), 1);
            else add_coh_i(cnt, 1);
        }
        return true;
    }
    bool ok = true;
    if (act) ok = fac_solve(x, sc, c, z, o);
    if (!hand) {
        if (act) fac_store(O, ld, v, o, 4);
        fac_vm0();
        if (!fac_agree(sm, ok)) return false;
        if (threadIdx.x == 0 && !quiet) fac_up(fac_flag(x, w, c), 4);
        return true;
    }
    const bool part = x.wc >= 3 && i >= 3;   // P(i, i - 1) and P(i, i) exist
    const int lane = fac_lane();
    double* X = &sm.tk.st[0][0][0];
    if (k.kind == FT_H1) {   // the strips exchanged through LDS
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int r = 0; r < 4; ++r) X[(v * 4 + p) * 256 + r * 64 + lane] = o[p][r];
    }
    if (!fac_agree(sm, ok)) return false;
    SchedDeps d;
    d.n = 0;
    if (part) deps_add(d, x.pp + i * (int64_t)4 + (k.kind == FT_H0 ? 1 : 0), 1);
    if (k.kind == FT_H0) {
        deps_add(d, x.pp + i * (int64_t)4 + 3, 1);
        deps_add(d, fac_flag(x, FacRow{i - 1}, c), 4);
    }
    if (!sched_wait_deps(sc, d, &sm.sh)) return false;
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = dbl4{0.0, 0.0, 0.0, 0.0};
    if (k.kind == FT_H0) {
        // block (i, i - 1) -= R (i - 1, i - 2)^T
        fac_store(O, b, v, o, 4);
        const double* A = uniform_ptr(fac_band(x, i - 1, c));
        O = fac_band(x, i, i - 1);
        const int li = lane & 15, lk = lane >> 4;
        uint32_t oa[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) oa[t] = lds_addr(sm.tk.st[0][0]) + 8u * (uint32_t)(lk * 64 + 16 * (t ^ lk) + li);
        fac_load(O, b, v, z, 4);
        if (LD == FAC_NARROW) fac_vm0();
#pragma unroll
        for (int q = 0; q < 4; ++q) fac_issue_a<LD>(A, b, q, sm.tk.st[q][0]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            fac_landed<LD, 2>(3 - q);
            fac_bar();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                dbl2 a[4];
                const uint32_t so = (uint32_t)q * (uint32_t)(2 * 16 * 64 * 8) + (uint32_t)h * (8 * 64 * 8);
                fac_read_a(oa[0] + so, oa[1] + so, oa[2] + so, oa[3] + so, a);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].x, o[q][2 * h], acc[t], 0, 0, 0);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].y, o[q][2 * h + 1], acc[t], 0, 0, 0);
            }
        }
        nt = 4;
    } else {
        // block (i, i) -= R R^T
        O = fac_band(x, i, i);
        nt = v + 1;
        fac_load(O, b, v, z, nt);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (t < nt) {
#pragma unroll
                for (int p = 0; p < 4; ++p)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(X[(t * 4 + p) * 256 + r * 64 + lane], o[p][r], acc[t], 0,
                                                                      0, 0);
            }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) z[t] -= acc[t];
    fac_store(O, b, v, z, nt);
    fac_vm0();
    fac_bar();
    if (threadIdx.x == 0 && !quiet) {
        fac_up(x.hx + i * (int64_t)2 + (k.kind == FT_H1 ? 1 : 0), 1);
        if (k.kind == FT_H0) fac_up(fac_flag(x, FacRow{i}, c), 4);
    }
    return true;
}

// ---------------------------------------------------------------------------
// The chain
// ---------------------------------------------------------------------------
// Wavefront S owns row tile S of the diagonal block (tiles z[t], t <= S, in
// registers) and strip S of the block below it, and factors panel S: the
// panel's 16 x 16 block goes from wavefront to wavefront only as Y_p in LDS,
// and the next wavefront has its own block up to date as soon as it has
// solved one tile with it.  The wavefronts meet through progress words in LDS
// rather than barriers, so a wavefront that is still busy with its strip does
// not hold up the others.
//
// What bounds it, in cycles at w 1,024 (29,400 per chunk): four pivots of
// 3,000 with a hand-over of about 1,500 between them, then the way of block
// row c + 1 out to H0(c + 2) and back (store, flag, poll, load: some 7,000).
// Eight wavefronts with 128 registers, four on the pivots and four on the
// strips, were slower (narrow 5.0 against 4.5 ms, w 1,024 21.9 against 19.0):
// the polls share LDS with the pivots.  Whole factors before and after the
// chain left barriers: nb 31,987 w 32 a 57 6.8 -> 4.5 ms, nb 100,000 w 1,024
// 26.9 -> 19.0 ms.

// Wait until every progress word e in [lo, hi) is at least a, and those in
// [lo2, hi2) at least b (one LDS read per poll).
__device__ inline bool ch_wait(const Sched& sc, FacSmem& sm, int lo, int hi, int a, int lo2 = 0, int hi2 = 0, int b = 0) {
    const int e = threadIdx.x & 31;
    const int need = e >= lo && e < hi ? a : (e >= lo2 && e < hi2 ? b : -1);
    int64_t t0 = -1;
    for (unsigned n = 0;; ++n) {
        if (__ballot(fac_lds_get(&sm.ch.w[e]) < need) == 0) break;
        if ((n & 255) == 255) {
            if (__builtin_amdgcn_readfirstlane(fac_lds_get(&sm.dead)) != 0) return false;
            if (__builtin_amdgcn_readfirstlane(ld_coh_i(sc.err)) != 0) return false;
            if (t0 < 0) t0 = wall_clock64();
            if (wall_clock64() - t0 > sc.spin_limit) {
                set_error_once(sc.err, STILES_ETIMEOUT);
                return false;
            }
        }
    }
    asm volatile("" ::: "memory");
    return true;
}
__device__ inline void ch_set(FacSmem& sm, int e, int v) {
    // LDS operations of one wavefront complete in order
    asm volatile("" ::: "memory");
    fac_lds_set(&sm.ch.w[e], v);
    asm volatile("" ::: "memory");
}
// Y Z^T for one tile (two chains of two products)
__device__ inline dbl4 ch_solve(const double* Y, const dbl4& z, int li, int lk) {
    double y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = Y[(4 * r + lk) * 17 + li];
    dbl4 p = dbl4{0.0, 0.0, 0.0, 0.0}, q = p;
    p = __builtin_amdgcn_mfma_f64_16x16x4f64(y[0], z[0], p, 0, 0, 0);
    q = __builtin_amdgcn_mfma_f64_16x16x4f64(y[1], z[1], q, 0, 0, 0);
    p = __builtin_amdgcn_mfma_f64_16x16x4f64(y[2], z[2], p, 0, 0, 0);
    q = __builtin_amdgcn_mfma_f64_16x16x4f64(y[3], z[3], q, 0, 0, 0);
    return p + q;
}
// sum over the four panels of A_p B_p^T, both operands in LDS or registers
template <class FA, class FB>
__device__ inline dbl4 ch_dot(FA&& a, FB&& b) {
    dbl4 e = dbl4{0.0, 0.0, 0.0, 0.0}, q = e;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        e = __builtin_amdgcn_mfma_f64_16x16x4f64(a(p, 0), b(p, 0), e, 0, 0, 0);
        q = __builtin_amdgcn_mfma_f64_16x16x4f64(a(p, 1), b(p, 1), q, 0, 0, 0);
        e = __builtin_amdgcn_mfma_f64_16x16x4f64(a(p, 2), b(p, 2), e, 0, 0, 0);
        q = __builtin_amdgcn_mfma_f64_16x16x4f64(a(p, 3), b(p, 3), q, 0, 0, 0);
    }
    return e + q;
}
#define CH_TILE(t, p) ((t) * ((t)-1) / 2 + (p))

// Row S of a diagonal block D: tiles t < S into z, the diagonal tile into zd,
// symmetric from its lower triangle.
__device__ inline void ch_load_row(const double* D, int b, int S, dbl4 (&z)[3], dbl4& zd) {
    const int lane = fac_lane(), li = lane & 15, lk = lane >> 4;
    D = uniform_ptr(D);
    b = fac_opaque(b);
#pragma unroll
    for (int t = 0; t < 3; ++t)
        if (t < S) {
#pragma unroll
            for (int r = 0; r < 4; ++r) z[t][r] = ld_coh_s(D, (uint32_t)((16 * S + li) + (16 * t + 4 * r + lk) * b));
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = imax_(li, 4 * r + lk), j = imin_(li, 4 * r + lk);
        zd[r] = ld_coh_s(D, (uint32_t)((16 * S + i) + (16 * S + j) * b));
    }
}
// One 16 x 16 tile (row tile i, column tile j) of the block at B to memory.
__device__ inline void ch_store(double* B, int b, int i, int j, const dbl4& v, int li, int lk) {
#pragma unroll
    for (int r = 0; r < 4; ++r) st_coh_s(B, (uint32_t)((16 * i + li) + (16 * j + 4 * r + lk) * b), v[r]);
}
__device__ inline void ch_put(double* X, const dbl4& v, int lane) {
#pragma unroll
    for (int r = 0; r < 4; ++r) X[r * 64 + lane] = v[r];
}
__device__ inline dbl4 ch_get(const double* X, int lane) {
    dbl4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = X[r * 64 + lane];
    return v;
}
// c += a b^T, the tiles in operand order
__device__ inline void ch_mma(dbl4& c, const dbl4& a, const dbl4& b) {
#pragma unroll
    for (int r = 0; r < 4; ++r) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], b[r], c, 0, 0, 0);
}

// One wavefront of the chain (S = its number).  The code is the same for all
// four, with S a run-time value, so that the chain's loop stays in the
// instruction cache: the tiles of a row are shifted down as they are used.
__device__ inline bool fac_chain_wave(const FacCtx& x, const Sched& sc, FacSmem& fs, int c0, int c1, int* info,
                                      bool quiet) {
    ChainSmem& sm = fs.ch;
    const int S = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = fac_lane(), li = lane & 15, lk = lane >> 4;
    const int b0 = x.L.b;
    dbl4 o[4];        // strip S of the block row below the previous chunk
    dbl4 z[3], zd;    // row S of the diagonal block: the tiles left of its own, its own
    dbl4 dd = dbl4{0.0, 0.0, 0.0, 0.0};   // what its own loses to the strip
    dbl4 y[4];        // strip S of the block row below this chunk
    int* pend_po = nullptr;   // flag to raise once this wavefront's stores are in memory
    bool have_z = false;
    for (int c = c0; c < c1; ++c) {
        const int b = fac_opaque(b0);
        double(&Yc)[4][16 * 17] = sm.Y[c & 1];
        double(&Lc)[6][256] = sm.Lt[c & 1];
        double* D = (double*)uniform_ptr(fac_band(x, c, c));
        const bool above = c > 0 && x.wc >= 1;        // there is a block row R of the chunk before
        const bool below = x.wc >= 1 && c + 1 < x.nc;
        const bool taken = x.wc >= 2 && c >= 1;       // block (c + 1, c) comes from H0(c + 1)
        double* Rb = below ? (double*)uniform_ptr(fac_band(x, c + 1, c)) : nullptr;
        const int* hx = x.hx + (c + 1) * (int64_t)2;
        // row S of the diagonal block, up to date with every chunk before c
        if (!have_z) {
            if (x.wc >= 2 && c >= 2 && !fac_wait1(sc, x.hx + c * (int64_t)2 + 1, 1)) return false;
            ch_load_row(D, b, S, z, zd);
        }
        have_z = false;
        zd -= dd;
        if (above) {
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                if (t >= S || (S == 3 && t > 0)) continue;   // tiles (3, 1) and (3, 2) by wavefront 0
                if (!ch_wait(sc, fs, CW_R + t, CW_R + t + 1, 4 * c)) return false;
                z[t] -= ch_dot([&](int p, int r) { return sm.R[t][p][r * 64 + lane]; }, [&](int p, int r) { return o[p][r]; });
            }
        }
        if (S > 0) ch_set(fs, CW_D + S, c + 1);
        if (S > 0 && pend_po) {   // what was stored during the last chunk
            fac_vm0();
            if (lane == 0 && !quiet) fac_up(pend_po, 1);
            pend_po = nullptr;
        }
        // panels before this wavefront's own
        for (int p = 0; p < S; ++p) {
            if (S == 3 && p > 0 && above) {
                if (p == 1 && !ch_wait(sc, fs, CW_X, CW_X + 1, c + 1)) return false;
                z[0] -= ch_get(sm.X[p - 1], lane);
            }
            if (!ch_wait(sc, fs, CW_Y + p, CW_Y + p + 1, c + 1)) return false;
            const dbl4 l = ch_solve(Yc[p], z[0], li, lk);
            ch_put(Lc[CH_TILE(S, p)], l, lane);
            ch_set(fs, CW_L + S, 4 * c + p + 1);
            const dbl4 m = -l;
            ch_mma(zd, m, l);
            if (p + 1 < S) {
                if (!ch_wait(sc, fs, CW_L + p + 1, CW_L + S, 4 * c + p + 1)) return false;
                ch_mma(z[1], ch_get(Lc[CH_TILE(p + 1, p)], lane), m);
                if (p + 2 < S) ch_mma(z[2], ch_get(Lc[CH_TILE(p + 2, p)], lane), m);
            }
            ch_store(D, b, S, p, l, li, lk);
            z[0] = z[1];
            z[1] = z[2];
        }
        // its own; whether the block below is ready is asked before and looked at after
        const int early = below && taken ? ld_coh_i(hx) : 1;
        {
            double l[4], yv[4];
            const int fail = f16_factor(zd, l, yv);
#pragma unroll
            for (int q = 0; q < 4; ++q) Yc[S][li * 17 + 4 * q + lk] = yv[q];
            ch_set(fs, CW_Y + S, c + 1);
            if (S == 0 && pend_po) {   // wavefront 0's row of the last chunk (it does not wait for its stores before)
                fac_vm0();
                if (lane == 0 && !quiet) fac_up(pend_po, 1);
            }
            ch_store(D, b, S, S, dbl4{l[0], l[1], l[2], l[3]}, li, lk);
            if (fail >= 0 && lane == 0)
                __hip_atomic_fetch_min((GLOBAL_AS int*)info, x.col0 + c * FC + 16 * S + fail + 1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            double* Yg = (double*)uniform_ptr(x.Yd + (int64_t)c * 1024 + S * 256);
#pragma unroll
            for (int r = 0; r < 4; ++r) st_coh_s(Yg, (uint32_t)(r * 64 + lane), Yc[S][(4 * r + lk) * 17 + li]);
        }
        const bool ready = __builtin_amdgcn_readfirstlane(early) != 0;
        if (below && ready) fac_load(Rb, b, S, y, 4);
        if (S == 0) {
            if (above) {   // for wavefront 3, which has the longest row
                if (!ch_wait(sc, fs, CW_R + 1, CW_R + 4, 4 * c)) return false;
#pragma unroll 1
                for (int t = 1; t < 3; ++t) {
                    const dbl4 d = ch_dot([&](int p, int r) { return sm.R[t][p][r * 64 + lane]; },
                                          [&](int p, int r) { return sm.R[3][p][r * 64 + lane]; });
                    ch_put(sm.X[t - 1], d, lane);
                }
                ch_set(fs, CW_X, c + 1);
            }
            ch_set(fs, CW_D + S, c + 1);
        }
        pend_po = x.po + c * (int64_t)4 + S;
        if (x.wc >= 2) {   // the tasks that the chain waits for need the row soon
            fac_vm0();
            if (lane == 0 && !quiet) fac_up(pend_po, 1);
            pend_po = nullptr;
        }
        // strip S of the block row below
        if (below) {
            if (!ready) {
                if (!fac_wait1(sc, hx, 1)) return false;
                fac_load(Rb, b, S, y, 4);
            }
            // the next diagonal block's row, if it is there too
            if (x.wc < 2 || c + 1 < 2 || __builtin_amdgcn_readfirstlane(ld_coh_i(hx + 1)) != 0) {
                ch_load_row(fac_band(x, c + 1, c + 1), b, S, z, zd);
                have_z = true;
            }
            dd = dbl4{0.0, 0.0, 0.0, 0.0};
            auto panel = [&](int p) {
                dbl4 lt[4];
#pragma unroll
                for (int t = p + 1; t < 4; ++t) lt[t] = ch_get(Lc[CH_TILE(t, p)], lane);
                o[p] = ch_solve(Yc[p], y[p], li, lk);
                const dbl4 m = -o[p];
#pragma unroll
                for (int t = p + 1; t < 4; ++t) ch_mma(y[t], lt[t], m);
                ch_mma(dd, o[p], o[p]);
            };
            if (__builtin_amdgcn_readfirstlane(fac_lds_get(&sm.w[CW_Y + 3])) >= c + 1) {
                // the last panel is there, so everything is: no waits between
                // the panels, the next one's operands on their way meanwhile
#pragma unroll
                for (int p = 0; p < 4; ++p) panel(p);
            } else {
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    // Y_p and the tiles below it
                    if (!ch_wait(sc, fs, CW_Y + p, CW_Y + p + 1, c + 1, CW_L + p + 1, CW_L + 4, 4 * c + p + 1)) return false;
                    panel(p);
                }
            }
            // the last chunk's strips have been read by every wavefront
            if (!ch_wait(sc, fs, CW_D, CW_D + 4, c + 1)) return false;
#pragma unroll
            for (int p = 0; p < 4; ++p) ch_put(sm.R[S][p], o[p], lane);
            ch_set(fs, CW_R + S, 4 * c + 4);
            if (S > 0) {
                // to memory, and wavefront 0's strip with wavefront 1's: that
                // one's next panel is what everything waits for
#pragma unroll
                for (int p = 0; p < 4; ++p) ch_store(Rb, b, S, p, o[p], li, lk);
                if (S == 1) {
                    if (!ch_wait(sc, fs, CW_R, CW_R + 1, 4 * c + 4)) return false;
#pragma unroll
                    for (int p = 0; p < 4; ++p) ch_store(Rb, b, 0, p, ch_get(sm.R[0][p], lane), li, lk);
                }
                fac_vm0();
                if (lane == 0) {
                    if (pend_po && !quiet) fac_up(pend_po, 1);
                    add_coh_i(fac_flag(x, FacRow{c + 1}, c), S == 1 ? 2 : 1);
                }
                pend_po = nullptr;
            }
        }
    }
    fac_vm0();
    if (lane == 0 && pend_po && !quiet) fac_up(pend_po, 1);
    return true;
}

// Chunks c0 .. c1 - 1 of one matrix, all of them or (with wc 0) one; false when
// the kernel must stop.
__device__ inline bool fac_chain(const FacCtx& x, const Sched& sc, FacSmem& sm, int c0, int c1, int* info, bool quiet) {
    __syncthreads();
    if (threadIdx.x < 32) sm.ch.w[threadIdx.x] = 0;
    __syncthreads();
    const bool ok = fac_chain_wave(x, sc, sm, c0, c1, info, quiet);
    fac_vm0();
    return fac_agree(sm, ok);
}
