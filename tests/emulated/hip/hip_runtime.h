// The part of HIP that the library uses, on the CPU, for tests: a thread of a workgroup is a fiber, a workgroup that runs
// beside others has an OS thread of its own (workgroup.cpp).  Device memory lies between inaccessible pages: against the one
// behind it, or, with EMULATED_ORDER set, against the one in front, so that in one of the two an access outside an allocation
// ends the process with the address (up to 15 bytes of rounding at the end excepted).  Not seen: an access that leaves its part
// of an allocation (a lane's, a channel's) or of the workgroup's LDS for another part.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <functional>
#include <tuple>

#define __device__
#define __global__
#define __host__
#define __shared__ thread_local
#define __forceinline__ inline
#define __align__(n) __attribute__((aligned(n)))
#define __launch_bounds__(...)
#define __restrict__

struct uint2 { uint32_t x, y; } __attribute__((aligned(8)));
struct uint3 { uint32_t x, y, z; };
struct uint4 { uint32_t x, y, z, w; } __attribute__((aligned(16)));
inline uint2 make_uint2(uint32_t a, uint32_t b) { return uint2{a, b}; }
inline uint4 make_uint4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return uint4{a, b, c, d}; }
struct dim3 { uint32_t x, y, z; dim3(uint32_t a = 1, uint32_t b = 1, uint32_t c = 1) : x(a), y(b), z(c) {} };
extern thread_local uint3 threadIdx, blockIdx, blockDim, gridDim;
using std::max;
using std::min;
inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
inline uint32_t __float_as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
inline int __popc(uint32_t v) { return __builtin_popcount(v); }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __ffsll(long long v) { return __builtin_ffsll(v); }
inline unsigned long long wall_clock64() { return 0; }

// ---- atomics ---------------------------------------------------------------------------------
#define EMULATED_ATOMICS(T)                                                                                        \
  inline T atomicAdd(T *p, T v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }                            \
  inline T atomicOr(T *p, T v) { return __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST); }                              \
  inline T atomicAnd(T *p, T v) { return __atomic_fetch_and(p, v, __ATOMIC_SEQ_CST); }                            \
  inline T atomicExch(T *p, T v) { return __atomic_exchange_n(p, v, __ATOMIC_SEQ_CST); }                          \
  inline T atomicCAS(T *p, T c, T v) {                                                                             \
    __atomic_compare_exchange_n(p, &c, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);                              \
    return c;                                                                                                      \
  }                                                                                                                \
  inline T atomicMin(T *p, T v) {                                                                                  \
    T o = __atomic_load_n(p, __ATOMIC_SEQ_CST);                                                                    \
    while (v < o && !__atomic_compare_exchange_n(p, &o, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)) {}          \
    return o;                                                                                                      \
  }                                                                                                                \
  inline T atomicMax(T *p, T v) {                                                                                  \
    T o = __atomic_load_n(p, __ATOMIC_SEQ_CST);                                                                    \
    while (v > o && !__atomic_compare_exchange_n(p, &o, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)) {}          \
    return o;                                                                                                      \
  }
EMULATED_ATOMICS(uint32_t)
EMULATED_ATOMICS(unsigned long long)
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)
#define __builtin_amdgcn_fence(...) __atomic_thread_fence(__ATOMIC_SEQ_CST)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
inline void __threadfence_block() { __atomic_thread_fence(__ATOMIC_SEQ_CST); }

// ---- what the threads of a wavefront or a workgroup do together --------------------------------
enum { OP_BALLOT = 1, OP_READLANE, OP_READFIRST, OP_DPP, OP_UP, OP_XOR, OP_BARRIER, OP_SLEEP, OP_BALLOT_HERE, OP_READLANE_HERE };
uint64_t together(int op, uint64_t v, uint64_t arg, uint64_t old = 0);
inline unsigned long long __ballot(int p) { return together(OP_BALLOT, p ? 1 : 0, 0); }
inline int __builtin_amdgcn_readlane(int v, int l) { return (int)together(OP_READLANE, (uint32_t)v, (uint64_t)l); }
inline int __builtin_amdgcn_readfirstlane(int v) { return (int)together(OP_READFIRST, (uint32_t)v, 0); }
inline int __builtin_amdgcn_update_dpp(int old, int v, int ctrl, int, int, bool) { return (int)together(OP_DPP, (uint32_t)v, (uint64_t)ctrl, (uint32_t)old); }
inline void __builtin_amdgcn_s_barrier() { together(OP_BARRIER, 0, 0); }
inline void __syncthreads() { together(OP_BARRIER, 0, 0); }
inline void __builtin_amdgcn_s_sleep(int) { together(OP_SLEEP, 0, 0); }
template <class T> inline T shuffled(int op, T v, int arg) {
  uint64_t u = 0;
  memcpy(&u, &v, sizeof(T));
  u = together(op, u, (uint64_t)arg);
  memcpy(&v, &u, sizeof(T));
  return v;
}
template <class T> inline T __shfl(T v, int l, int) { return shuffled(OP_READLANE, v, l); }
template <class T> inline T __shfl_up(T v, int d, int) { return shuffled(OP_UP, v, d); }
template <class T> inline T __shfl_xor(T v, int d, int) { return shuffled(OP_XOR, v, d); }

// The same for the lanes of a wavefront that have come to a place in a branch: those that wait there with the same key.
inline unsigned long long ballot_here(int p, const void *key) { return together(OP_BALLOT_HERE, p ? 1 : 0, 0, (uint64_t)key); }
template <class T> inline T readlane_here(T v, int l, const void *key) { return (T)together(OP_READLANE_HERE, (uint64_t)v, (uint64_t)l, (uint64_t)key); }

// ---- the host's side: everything happens at once ------------------------------------------------
typedef int hipError_t;
typedef struct emulated_stream *hipStream_t;
typedef struct emulated_event *hipEvent_t;
enum { hipSuccess = 0, hipErrorNotReady = 600 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum { hipDeviceAttributeMultiprocessorCount, hipEventDisableTiming, hipStreamNonBlocking };
hipError_t hipMalloc(void **p, size_t n);
hipError_t hipFree(void *p);
inline hipError_t hipHostMalloc(void **p, size_t n) { return hipMalloc(p, n); }
inline hipError_t hipHostFree(void *p) { return hipFree(p); }
inline hipError_t hipHostGetDevicePointer(void **d, void *h, int) { *d = h; return 0; }
inline hipError_t hipGetLastError() { return 0; }
inline hipError_t hipGetDevice(int *d) { *d = 0; return 0; }
inline hipError_t hipDeviceGetAttribute(int *v, int, int) { *v = 24; return 0; }
inline hipError_t hipDeviceSynchronize() { return 0; }
inline hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return 0; }
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return 0; }
inline hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return 0; }
inline hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { memset(d, v, n); return 0; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return 0; }
inline hipError_t hipStreamQuery(hipStream_t) { return 0; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, int) { *s = nullptr; return 0; }
inline hipError_t hipStreamDestroy(hipStream_t) { return 0; }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, int) { return 0; }
inline hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return 0; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, int) { *e = nullptr; return 0; }
inline hipError_t hipEventDestroy(hipEvent_t) { return 0; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return 0; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return 0; }
inline hipError_t hipEventQuery(hipEvent_t) { return 0; }
inline hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0; return 0; }
#define HIP_SYMBOL(x) x
template <class T> inline hipError_t hipGetSymbolAddress(void **p, T &x) { *p = (void *)&x; return 0; }

// kernels whose name says that their workgroups wait for each other run all of them at once
void run_grid(dim3 grid, dim3 block, bool at_once, const std::function<void()> &fn);
template <class... A, class... B> void launch(void (*kernel)(A...), const char *name, dim3 grid, dim3 block, B... args) {
  const std::tuple<A...> t(args...);
  run_grid(grid, block, strstr(name, "true") != nullptr, [=]() { std::apply(kernel, t); });
}
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) launch(kernel, #kernel, grid, block, __VA_ARGS__)
