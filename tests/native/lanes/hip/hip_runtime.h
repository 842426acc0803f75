// One wave of 64 threads on the CPU: enough of the device language to run the
// time-sliced finder's window functions (hough_tw.h) lane by lane. Every lane is a
// thread; the wave's exchanges (ballot, readlane, shuffles) meet at a barrier.
#pragma once

#include <barrier>
#include <climits>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>

#define __host__
#define __device__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define asm
#define volatile(...)

typedef int hipError_t;
typedef struct ihipStream_t *hipStream_t;
struct float2 {
    float x, y;
};
struct Index3 {
    unsigned x, y, z;
};
inline thread_local Index3 threadIdx;
inline Index3 blockIdx;

namespace lanes {
inline std::barrier<> meet(64);
inline uint64_t word[64];
template <class T>
T from(T v, int l) {   // lane l's v
    static_assert(sizeof(T) <= 8);
    std::memcpy(&word[threadIdx.x & 63], &v, sizeof v);
    meet.arrive_and_wait();
    T r;
    std::memcpy(&r, &word[l & 63], sizeof r);
    meet.arrive_and_wait();
    return r;
}
}  // namespace lanes

inline unsigned long long __ballot(bool p) {
    lanes::word[threadIdx.x & 63] = p;
    lanes::meet.arrive_and_wait();
    unsigned long long m = 0;
    for (int i = 0; i < 64; ++i) m |= (unsigned long long)(lanes::word[i] & 1) << i;
    lanes::meet.arrive_and_wait();
    return m;
}
inline void __syncthreads() { lanes::meet.arrive_and_wait(); }
template <class T>
T __shfl_up(T v, int o, int) {
    const int me = (int)(threadIdx.x & 63);
    return lanes::from(v, me >= o ? me - o : me);
}
inline int __popcll(unsigned long long m) { return __builtin_popcountll(m); }
template <class T>
T min(T a, T b) { return b < a ? b : a; }
template <class T>
T max(T a, T b) { return a < b ? b : a; }
template <class To, class From>
To bits(From v) {
    To r;
    std::memcpy(&r, &v, sizeof r);
    return r;
}
inline float __int_as_float(int v) { return bits<float>(v); }
inline int __float_as_int(float v) { return bits<int>(v); }
inline unsigned __float_as_uint(float v) { return bits<unsigned>(v); }
template <class T, class U>
T atomicAdd(T *p, U v) { return __atomic_fetch_add(p, v, __ATOMIC_RELAXED); }
template <class T>
T atomicMin(T *p, T v) {
    T old = __atomic_load_n(p, __ATOMIC_RELAXED);
    while (v < old && !__atomic_compare_exchange_n(p, &old, v, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED)) {
    }
    return old;
}
inline unsigned long long wall_clock64() { return 0; }

#define __builtin_amdgcn_readfirstlane(v) (v)   // of values that every lane holds
#define __builtin_amdgcn_readlane(v, l) lanes::from((v), (l))
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rows, banks, bound) ((void)(ctrl), (void)(rows), (v))   // not run here
#define __builtin_amdgcn_fence(order, scope) __atomic_thread_fence(__ATOMIC_SEQ_CST)
