// Device helpers shared by the kernels' translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scan {
namespace {

__device__ __forceinline__ uint8_t ld_u8(const uint8_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_u8(uint8_t* p, uint8_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t ld_i32(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_i32(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Union-find with min-id hooking: a root is only ever linked below a smaller
// root, so parent[x] <= x always holds, no cycle can form, and the final root
// of every tree is its minimum member.  find() halves paths; every value it
// writes is an ancestor of x, which stays an ancestor forever.
__device__ int32_t uf_find(int32_t* parent, int32_t x) {
  while (true) {
    const int32_t p = ld_i32(parent + x);
    if (p == x) return x;
    const int32_t gp = ld_i32(parent + p);
    if (gp == p) return p;
    st_i32(parent + x, gp);
    x = gp;
  }
}

__device__ void uf_union(int32_t* parent, int32_t a, int32_t b) {
  while (true) {
    a = uf_find(parent, a);
    b = uf_find(parent, b);
    if (a == b) return;
    if (a > b) { int32_t t = a; a = b; b = t; }
    const int32_t old = atomicCAS(parent + b, b, a);
    if (old == b) return;
  }
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long x) {
  for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
  return x;
}

}  // namespace
}  // namespace scan
