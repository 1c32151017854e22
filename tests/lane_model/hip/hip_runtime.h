// Host declarations for compiling the device headers' scalar helpers as plain C++ (tests
// only): a lane is a host thread of control, and each compare-and-swap is a point where
// the other lanes of the wavefront get their turn (probe.cpp).
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <cmath>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static

struct dim3 {
    unsigned x, y, z;
};
extern dim3 threadIdx, blockIdx, blockDim, gridDim;
void __syncthreads();

typedef int hipError_t;
typedef void *hipStream_t;
enum { hipSuccess = 0 };
const char *hipGetErrorString(hipError_t);

struct uint2 {
    uint32_t x, y;
};
struct uint4 {
    uint32_t x, y, z, w;
};
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
inline double __hiloint2double(int hi, int lo) {
    const uint64_t b = ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
    double d;
    memcpy(&d, &b, 8);
    return d;
}
inline float __uint_as_float(uint32_t u) {
    float f;
    memcpy(&f, &u, 4);
    return f;
}
inline uint32_t __float_as_uint(float f) {
    uint32_t u;
    memcpy(&u, &f, 4);
    return u;
}

void other_lanes();  // runs the wavefront's other lanes up to their next such point
inline int32_t atomicCAS(int32_t *p, int32_t expect, int32_t v) {
    other_lanes();
    const int32_t was = *p;
    if (was == expect) *p = v;
    return was;
}
template <typename T, typename U>
T atomicAdd(T *p, U v) {
    const T was = *p;
    *p += (T)v;
    return was;
}

inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline long long __double_as_longlong(double d) {
    long long b;
    memcpy(&b, &d, 8);
    return b;
}

// wave operations: defined by the models that need them
int __lane_id();
uint64_t __ballot(int);
uint32_t mask_bits_below(uint64_t mask);
template <typename T>
T __shfl_xor(T, int, int = 64);
template <typename T>
T __shfl_up(T, int, int = 64);
template <typename T>
T __shfl(T, int, int = 64);
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)0)
#define __builtin_amdgcn_s_setprio(p) ((void)0)
#define __builtin_amdgcn_mbcnt_hi(m, below) (mask_bits_below((uint64_t)(m) << 32) + (below))
#define __builtin_amdgcn_mbcnt_lo(m, below) (mask_bits_below((uint64_t)(m)) + (below))
#define __atomic_load_n(p, order) (*(p))
#define __HIP_MEMORY_SCOPE_SYSTEM 0
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))
