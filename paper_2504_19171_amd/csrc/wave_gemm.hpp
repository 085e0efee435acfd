// Building blocks of the FP64 products of Phase 2: operands that go straight
// into LDS (global_load_lds_dwordx4: lane l's 16 bytes land at 16 l from the
// instruction's base, 1 KB per instruction; no registers hold data in flight),
// and the sum of the wavefronts' partial blocks.
//
// v_mfma_f64_16x16x4_f64 lane layout (lane l): A[l%16][l/16], B[l/16][l%16],
// D element r = D[4r + l/16][l%16].
#pragma once
#include "common.hpp"

typedef __attribute__((address_space(3))) void lds_void_t;

// LDS byte address of a pointer into LDS.
__device__ inline uint32_t lds_addr(const double* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) double*)p;
}

// An operand of 16 k contiguous along k: element (x, k) lies at [x * 16 +
// 2 ((k / 2) ^ (x % 8)) + k % 2], so that what 16 rows and four pairs of k take
// falls in different banks.  wg_lane: where in the operand lane l's pair of a
// kilobyte load begins (rows x = 8 i + l / 8 for load i); wg_at: the byte offset
// of the pair k = 2 (l / 16) of row x (k + 8: the offset ^ 64).
__device__ __forceinline__ uint32_t wg_lane(int ld, int i) {
    const int l = threadIdx.x & 63;
    return (uint32_t)(2 * ((l & 7) ^ (l >> 3)) + (8 * i + (l >> 3)) * ld);
}
__device__ __forceinline__ uint32_t wg_at(int x) {
    const int lk = (threadIdx.x & 63) >> 4;
    return (uint32_t)(x * 16 + 2 * (lk ^ (x & 7))) * 8u;
}

// Operands of 16 k for one wavefront: a[i][m], b[i][m] hold k = 8 m + 2 (l / 16)
// and the next one, of row (column) l % 16 of tile i.  Reads and their wait in
// one block, as the compiler would also wait for every load into LDS still in
// flight.  wg_read_kk: both along k (addresses wg_at); wg_read_xk: a along x,
// rows of 64, the addresses those of k = 2 (l / 16).
typedef double wg2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void wg_read_kk(uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1, wg2 (&a)[2][2], wg2 (&b)[2][2]) {
    const uint32_t a0m = a0 ^ 64, a1m = a1 ^ 64, b0m = b0 ^ 64, b1m = b1 ^ 64;
    asm volatile(
        "ds_read_b128 %0, %8\n\t"
        "ds_read_b128 %4, %12\n\t"
        "ds_read_b128 %5, %13\n\t"
        "ds_read_b128 %1, %9\n\t"
        "ds_read_b128 %2, %10\n\t"
        "ds_read_b128 %6, %14\n\t"
        "ds_read_b128 %7, %15\n\t"
        "ds_read_b128 %3, %11\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a[0][0]), "=&v"(a[1][0]), "=&v"(a[0][1]), "=&v"(a[1][1]), "=&v"(b[0][0]), "=&v"(b[1][0]), "=&v"(b[0][1]),
          "=&v"(b[1][1])
        : "v"(a0), "v"(a1), "v"(a0m), "v"(a1m), "v"(b0), "v"(b1), "v"(b0m), "v"(b1m)
        : "memory");
}
__device__ __forceinline__ void wg_read_xk(uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1, wg2 (&a)[2][2], wg2 (&b)[2][2]) {
    const uint32_t b0m = b0 ^ 64, b1m = b1 ^ 64;
    asm volatile(
        "ds_read2st64_b64 %0, %8 offset1:1\n\t"
        "ds_read_b128 %4, %10\n\t"
        "ds_read_b128 %5, %11\n\t"
        "ds_read2st64_b64 %1, %9 offset1:1\n\t"
        "ds_read2st64_b64 %2, %8 offset0:8 offset1:9\n\t"
        "ds_read_b128 %6, %12\n\t"
        "ds_read_b128 %7, %13\n\t"
        "ds_read2st64_b64 %3, %9 offset0:8 offset1:9\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a[0][0]), "=&v"(a[1][0]), "=&v"(a[0][1]), "=&v"(a[1][1]), "=&v"(b[0][0]), "=&v"(b[1][0]), "=&v"(b[0][1]),
          "=&v"(b[1][1])
        : "v"(a0), "v"(a1), "v"(b0), "v"(b1), "v"(b0m), "v"(b1m)
        : "memory");
}

// ---------------------------------------------------------------------------
// 32 x 32 block by a whole workgroup, the sum spread over its wavefronts
// ---------------------------------------------------------------------------
// For blocks whose latency counts.  The sum is cut into eight pieces, one or two
// per wavefront, and the partial blocks are added in a fixed order, the same
// for either number, so results depend neither on timing nor on the workgroup.

// One term: A(i, k) = a[k + i lda] (read device-coherent), B(k, j) = b[k + j
// ldb], i, j < 32, k < K (a multiple of 16).
struct Seg {
    const double* a;
    const double* b;
    int lda, ldb, K;
};
#define WG_PIECES 8
#define WG_CHUNK (2 * 32 * 16)      // doubles: 16 k of A, then of B
#define WG_WAVE (2 * WG_CHUNK)      // a wavefront's staging: two chunks

// s_waitcnt immediates, gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt in
// 6:4, lgkmcnt in 11:8; a counter at its maximum is not waited for.
#define WG_VMCNT8 0x0F78
#define WG_VMCNT4 0x0F74
#define WG_VMCNT0 0x0F70

// acc0 (and acc1, with four wavefronts) += this wavefront's piece(s) w (and w +
// 4) of the terms 0 .. nseg - 1 (seg(q)) of total length ktot, cut at multiples
// of 16.  sw: its WG_WAVE doubles of LDS.  The chunks of all its terms and
// pieces are one stream, two in flight; the vmcnt waits assume no other memory
// access of this wavefront in between (loads issued before are older and
// complete first).
// gate(pre) waits until A may be read, false if it never may; pre() issues the
// first loads of B meanwhile (B lies farther away than A, which has just been
// written).
template <int NW, class F, class G>
__device__ __forceinline__ bool wave_sum(dbl4 (&acc0)[2][2], dbl4 (&acc1)[2][2], int nseg, int ktot, double* sw, F&& seg,
                                         G&& gate) {
    if (NW < 8 && !gate([]() {})) return false;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = threadIdx.x & 15;
    const int per = 16 * (((ktot >> 4) + WG_PIECES - 1) / WG_PIECES);
    const uint32_t s0 = lds_addr(sw);
    const uint32_t r0 = wg_at(li), r1 = wg_at(li + 16);
    // the next chunk to issue: piece, its k up to ke, the term and where it starts
    int pc = w, k = imin_(per * w, ktot), ke = imin_(per * (w + 1), ktot), q = -1, t0 = 0, t1 = 0;
    const double *pa = nullptr, *pb = nullptr;
    uint32_t oa[4], ob[4];
    int left = 0, wr = 0, rd = 0;
    unsigned second = 0;   // bit i: the i-th chunk in flight is of the second piece
    auto there = [&]() {   // is there a chunk at k (of the next piece, if this one is done)
        if (k >= ke) {
            if (pc + NW >= WG_PIECES) return false;
            pc += NW;
            k = imin_(per * pc, ktot);
            ke = imin_(per * (pc + 1), ktot);
            if (k >= ke) return false;
        }
        if (k >= t1) {
            int K = 0;
            Seg g;
            do {
                t0 = t1;
                g = seg(++q);
                K = g.K;
                t1 = t0 + K;
            } while (k >= t1);
            pa = uniform_ptr(g.a);
            pb = uniform_ptr(g.b);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                oa[i] = wg_lane(g.lda, i) << 3;
                ob[i] = wg_lane(g.ldb, i) << 3;
            }
        }
        return true;
    };
    auto load_a = [&](int at, int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_global_load_lds((const void*)((const char*)(pa + (at - t0)) + oa[i]),
                                             (lds_void_t*)(sw + buf * WG_CHUNK + 128 * i), 16, 0, 16);
    };
    auto load_b = [&](int at, int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_global_load_lds((const void*)((const char*)(pb + (at - t0)) + ob[i]),
                                             (lds_void_t*)(sw + buf * WG_CHUNK + 512 + 128 * i), 16, 0, 0);
    };
    auto issued = [&]() {
        if (NW < 8) second |= (unsigned)(pc >= NW) << left;
        ++left;
        wr ^= 1;
        k += 16;
    };
    auto issue = [&]() {
        if (!there()) return;
        load_a(k, wr);
        load_b(k, wr);
        issued();
    };
    // with eight wavefronts: chunks whose B is on its way (the second only
    // beside the first).  (With four the CU's other workgroup has work for the
    // time: 64 matrices 17.6 ms without, 19.4 with.)
    int early = 0;
    if (NW == 8 && !gate([&]() {
            if (!there()) return;
            load_b(k, 0);
            early = 1;
            if (k + 16 >= imin_(ke, t1)) return;
            load_b(k + 16, 1);
            early = 2;
        })) {
        __builtin_amdgcn_s_waitcnt(WG_VMCNT0);   // no load into LDS outlives the workgroup
        return false;
    }
    if (NW == 8) early = __builtin_amdgcn_readfirstlane(early);
    if (NW == 8 && early > 0) {
        load_a(k, 0);
        issued();
        if (early > 1) {
            load_a(k, 1);
            issued();
        } else {
            issue();
        }
    } else if (NW < 8) {
        issue();
        issue();
    }
    while (left > 0) {
        if (left == 1) __builtin_amdgcn_s_waitcnt(WG_VMCNT0);
        else if (NW == 8 && early > 1) __builtin_amdgcn_s_waitcnt(WG_VMCNT4);   // only the second chunk's A is younger
        else __builtin_amdgcn_s_waitcnt(WG_VMCNT8);
        early = 0;
        __builtin_amdgcn_wave_barrier();
        wg2 a[2][2], b[2][2];
        const uint32_t st = s0 + (uint32_t)rd * (WG_CHUNK * 8u);
        wg_read_kk(st + r0, st + r1, st + 4096u + r0, st + 4096u + r1, a, b);
        const bool two = NW < 8 && (second & 1);
        second >>= 1;
        --left;
        rd ^= 1;
        issue();   // into the buffer just read
        auto mma = [&](dbl4 (&acc)[2][2]) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][m].x, b[j][m].x, acc[i][j], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][m].y, b[j][m].y, acc[i][j], 0, 0, 0);
            }
        };
        if (!two) mma(acc0);
        else mma(acc1);
    }
    return true;
}

#define WR_LD 33
#define WR_DOUBLES (32 * WR_LD)   // one wavefront's block in LDS

// Sum the wavefronts' accumulators into red[j*WR_LD + i] (column-major 32 x
// 32): pieces (0 + 4) + (1 + 5) + ... (with four wavefronts each has added its
// two).  smem (NW WR_DOUBLES, which may be the staging area of wave_sum) must
// not overlap red.  Ends with a barrier.
template <int NW>
__device__ inline void wave_reduce(const dbl4 (&acc)[2][2], double* smem, double* red) {
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    double* mine = smem + w * WR_DOUBLES;
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                mine[(tj * 16 + (l & 15)) * WR_LD + ti * 16 + 4 * r + (l >> 4)] = acc[ti][tj][r];
    __syncthreads();
    for (int e = threadIdx.x; e < 1024; e += 64 * NW) {
        const int o = (e >> 5) * WR_LD + (e & 31);
        double v = 0.0;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            double x = smem[p * WR_DOUBLES + o];
            if (NW == 8) x += smem[(p + 4) * WR_DOUBLES + o];
            v = p == 0 ? x : v + x;
        }
        red[o] = v;
    }
    __syncthreads();
}
