// Stand-in for the HIP runtime header: device code of the scheduler compiled for
// the host, a workgroup as one host thread per wavefront (its lane 0).
// Wavefront `emu_late` is held up before every value it broadcasts, i.e. before
// it reads a word that the workgroup shares.
#pragma once
#include <pthread.h>
#include <stdint.h>
#include <chrono>
#include <cmath>
#include <thread>

#define __device__
#define __host__
#define __global__
#define __HIP_MEMORY_SCOPE_AGENT 0

struct EmuIdx {
    unsigned x;
};
inline thread_local EmuIdx threadIdx;
inline pthread_barrier_t emu_barrier;
inline int emu_late = -1;
inline int* emu_raise = nullptr;   // a word that becomes 1 with its first read

inline void __syncthreads() { pthread_barrier_wait(&emu_barrier); }
inline void emu_hold() {
    if ((int)(threadIdx.x / 64) == emu_late) std::this_thread::sleep_for(std::chrono::milliseconds(50));
}
template <class F>
auto emu_broadcast(F f) {
    emu_hold();
    return f();
}
#define __builtin_amdgcn_readfirstlane(x) emu_broadcast([&] { return (x); })
#define __builtin_amdgcn_s_sleep(n) std::this_thread::yield()
#define __builtin_amdgcn_s_waitcnt(n) ((void)0)
#define __shfl_xor(x, o) (x)

template <class T>
T emu_load(const T* p) {
    T v;
    __atomic_load(p, &v, __ATOMIC_SEQ_CST);
    if ((const void*)p == emu_raise) {
        int up = 1;
        __atomic_store(emu_raise, &up, __ATOMIC_SEQ_CST);
    }
    return v;
}
template <class T>
void emu_store(T* p, T v) { __atomic_store(p, &v, __ATOMIC_SEQ_CST); }
#define __hip_atomic_load(p, order, scope) emu_load(p)
#define __hip_atomic_store(p, v, order, scope) emu_store(p, v)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_compare_exchange_strong(p, e, v, o1, o2, scope) \
    __atomic_compare_exchange_n(p, e, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)

inline int64_t wall_clock64() { return std::chrono::steady_clock::now().time_since_epoch().count(); }

// asm volatile(...): register hints, of no meaning here
#define asm
#define volatile(...)
