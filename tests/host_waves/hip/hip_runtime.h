// Runs kernels on the CPU, one workgroup at a time, wave by wave (see waves.cpp):
// just the names that bitmap.hip and the headers it includes use.  For tests of
// the order of accesses inside a workgroup; nothing of the library is built on it.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <functional>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct uint4 {
    unsigned x, y, z, w;
};
extern dim3 threadIdx, blockIdx, gridDim;

// ------------------------------------------------------------ waves and workgroups (waves.cpp)

void launch(dim3 grid, dim3 block, size_t lds, const std::function<void()>& kernel);
void workgroup_barrier();
void wait_forever();                                   // a wait for a workgroup that has not run
const uint64_t* exchange(uint64_t v);                  // every lane of the wave gives v: the wave's 64 values

#define hipLaunchKernelGGL(kernel, grid, block, lds, st, ...) \
    launch(grid, block, lds, [&] { (kernel)(__VA_ARGS__); })

inline void __syncthreads() { workgroup_barrier(); }
inline int __lane_id() { return (int)(threadIdx.x & 63); }
template <typename T>
T __shfl(T v, int src, int) { return (T)exchange((uint64_t)v)[src & 63]; }
template <typename T>
T __shfl_up(T v, int d, int) {
    const int l = __lane_id();
    return (T)exchange((uint64_t)v)[l >= d ? l - d : l];
}
inline uint64_t __ballot(bool p) {
    const uint64_t* x = exchange(p);
    uint64_t m = 0;
    for (int i = 0; i < 64; i++) m |= x[i] ? 1ull << i : 0;
    return m;
}
inline int __any(bool p) { return __ballot(p) != 0; }
inline int amdgcn_readlane(int v, int l) { return (int)exchange((uint32_t)v)[l]; }
// Row shifts right by 1 to 15, and lane 15 of a row or lane 31 to the rows after it;
// lanes without a source, or in a row that is masked out, keep `old`.
inline int amdgcn_update_dpp(int old, int v, int ctrl, int rows, int, bool) {
    const uint64_t* x = exchange((uint32_t)v);
    const int l = __lane_id();
    if (!(rows >> (l / 16) & 1)) return old;
    if (ctrl == 0x142) return l >= 16 ? (int)x[l / 16 * 16 - 1] : old;
    if (ctrl == 0x143) return l >= 32 ? (int)x[31] : old;
    const int n = ctrl - 0x110;
    return l % 16 >= n ? (int)x[l - n] : old;
}
#define __builtin_amdgcn_readlane amdgcn_readlane
#define __builtin_amdgcn_update_dpp amdgcn_update_dpp
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)exchange(0))
#define __builtin_amdgcn_s_sleep(n) wait_forever()

// ------------------------------------------------------------ arithmetic, atomics

inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline int __ffsll(uint64_t x) { return __builtin_ffsll((long long)x); }
inline uint64_t __umul64hi(uint64_t a, uint64_t b) { return (uint64_t)((unsigned __int128)a * b >> 64); }
template <typename T>
T swapped(T* p, T v) { const T was = *p; *p = v; return was; }
inline unsigned atomicAdd(unsigned* p, unsigned v) { return swapped(p, *p + v); }
inline unsigned atomicOr(unsigned* p, unsigned v) { return swapped(p, *p | v); }
inline unsigned atomicAnd(unsigned* p, unsigned v) { return swapped(p, *p & v); }
inline int atomicMax(int* p, int v) { return swapped(p, std::max(*p, v)); }
inline unsigned atomicCAS(unsigned* p, unsigned a, unsigned v) { return swapped(p, *p == a ? v : *p); }
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))

// ------------------------------------------------------------ host runtime: no device, nothing to do

enum hipError_t { hipSuccess, hipErrorOutOfMemory };
typedef void *hipStream_t, *hipEvent_t, *hipGraphExec_t;
enum { hipHostMallocDefault, hipFuncAttributeMaxDynamicSharedMemorySize };
template <typename T>
hipError_t hipMalloc(T**, size_t) { return hipErrorOutOfMemory; }
template <typename T>
hipError_t hipHostMalloc(T**, size_t, int) { return hipErrorOutOfMemory; }
inline hipError_t hipFree(void*) { return hipSuccess; }
inline hipError_t hipHostFree(void*) { return hipSuccess; }
inline hipError_t hipGetDevice(int*) { return hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void*, int, int) { return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return ""; }
