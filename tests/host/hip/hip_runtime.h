// Host stand-in for hip/hip_runtime.h: enough of it to compile the kernel headers for the CPU,
// so that tests can run device functions on host threads with their buffers behind guard
// pages.  A workgroup is one std::thread per lane; __syncthreads meets a barrier.  Wave
// intrinsics are declared only: what calls them cannot be linked.
#pragma once
#include <stdint.h>

#include <barrier>
#include <cmath>
#include <cstring>

#define __device__
#define __host__
#define __global__
#define __shared__
#define __forceinline__ inline
#define __noinline__
#define __align__(n) __attribute__((aligned(n)))
#define __launch_bounds__(...)
#define __HIP_MEMORY_SCOPE_AGENT 4
#define __HIP_MEMORY_SCOPE_SYSTEM 5

struct dim3 { unsigned x = 1, y = 1, z = 1; };
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
struct int2 { int32_t x, y; };
struct float2 { float x, y; };
struct double2 { double x, y; };
inline double2 make_double2(double x, double y) { return {x, y}; }
inline float2 make_float2(float x, float y) { return {x, y}; }

inline thread_local dim3 threadIdx, blockIdx;
inline dim3 gridDim, blockDim;
inline std::barrier<>* host_barrier;
inline void __syncthreads() { host_barrier->arrive_and_wait(); }

inline int __popc(uint32_t v) { return __builtin_popcount(v); }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline int __ffs(int v) { return __builtin_ffs(v); }
inline int __mul24(int a, int b) { return a * b; }
inline uint64_t __double_as_longlong(double v) { uint64_t u; std::memcpy(&u, &v, 8); return u; }
inline double __longlong_as_double(uint64_t u) { double v; std::memcpy(&v, &u, 8); return v; }
using std::fma;
using std::fmax;
using std::isfinite;
using std::ldexp;

template <class T, class U> T atomicOr(T* p, U v) { return __atomic_fetch_or(p, (T)v, __ATOMIC_RELAXED); }
template <class T, class U> T atomicAdd(T* p, U v);
template <class T> T __shfl(T, int, int = 64);
template <class T> T __shfl_xor(T, int, int = 64);

typedef uint32_t host_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t host_u32x2 __attribute__((ext_vector_type(2)));

// Raw buffers.  A load is out of range by the thread's offset alone: the narrower of the two
// readings of the range check (the other counts the uniform offset too).
struct __amdgpu_buffer_rsrc_t { char* base; int bytes; };
inline __amdgpu_buffer_rsrc_t __builtin_amdgcn_make_buffer_rsrc(void* p, int, int bytes, int) { return {(char*)p, bytes}; }
inline host_u32x4 __builtin_amdgcn_raw_buffer_load_b128(__amdgpu_buffer_rsrc_t r, int voff, int soff, int) {
  host_u32x4 v = {0, 0, 0, 0};
  if ((int64_t)voff + 16 <= r.bytes) std::memcpy(&v, r.base + voff + soff, 16);
  return v;
}
inline void __builtin_amdgcn_raw_buffer_store_b32(uint32_t v, __amdgpu_buffer_rsrc_t r, int voff, int soff, int) {
  if ((int64_t)voff + 4 <= r.bytes) std::memcpy(r.base + voff + soff, &v, 4);
}
inline void __builtin_amdgcn_raw_buffer_store_b64(host_u32x2 v, __amdgpu_buffer_rsrc_t r, int voff, int soff, int) {
  if ((int64_t)voff + 8 <= r.bytes) std::memcpy(r.base + voff + soff, &v, 8);
}

inline uint32_t __builtin_amdgcn_readfirstlane(uint32_t v) { return v; }   // of values all lanes hold
inline void __builtin_amdgcn_fence(int, const char*, ...) {}
inline void __builtin_amdgcn_s_barrier() { __syncthreads(); }
inline void __builtin_amdgcn_sched_barrier(int) {}

// The data-parallel moves of the kernels, through a table of the workgroup's lanes.
inline int host_lanes[1024];
inline int __builtin_amdgcn_mov_dpp(int v, int ctrl, int, int, bool) {
  const unsigned t = threadIdx.x;
  host_lanes[t] = v;
  __syncthreads();
  const unsigned from = ctrl == 0xB1 ? t ^ 1 : ctrl == 0x4E ? t ^ 2 : ctrl == 0x141 ? t ^ 7 : t ^ 15;
  const int r = host_lanes[from];
  __syncthreads();
  return r;
}

int __builtin_amdgcn_perm(uint32_t, uint32_t, uint32_t);
int __builtin_amdgcn_ds_bpermute(int, int);
int __builtin_amdgcn_ds_swizzle(int, int);
template <class V> V __builtin_amdgcn_mfma_i32_16x16x64_i8(V, V, V, int, int, int);
