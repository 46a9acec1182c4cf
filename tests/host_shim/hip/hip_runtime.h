// Stand-in for the HIP runtime header, so that device functions can be compiled
// for the host and run one lane at a time under the address sanitizer.  It
// keeps every index, load and store; what waits for other lanes does nothing
// and what exchanges values with them returns the lane's own, so results mean
// nothing and only addresses do.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>

#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __align__(n) __attribute__((aligned(n)))
#define __forceinline__ inline
#define __noinline__ __attribute__((noinline))
#define __launch_bounds__(...)
#define __HIP_MEMORY_SCOPE_AGENT 0

struct uint3_ {
  unsigned x, y, z;
};
inline uint3_ threadIdx{0, 0, 0}, blockIdx{0, 0, 0}, blockDim{256, 1, 1}, gridDim{1, 1, 1};
struct alignas(16) double2 {
  double x, y;
};
struct alignas(8) uint2 {
  unsigned x, y;
};
struct alignas(8) float2 {
  float x, y;
};
struct alignas(16) uint4 {
  unsigned x, y, z, w;
};
struct alignas(16) float4 {
  float x, y, z, w;
};

template <typename A, typename B>
constexpr std::common_type_t<A, B> min(A a, B b) {
  return b < a ? b : a;
}
template <typename A, typename B>
constexpr std::common_type_t<A, B> max(A a, B b) {
  return a < b ? b : a;
}
inline void __syncthreads() {}
template <typename T>
T __shfl(T v, int) {
  return v;
}
template <typename T>
T __shfl_xor(T v, int) {
  return v;
}
inline unsigned long long __ballot(bool) { return 0ull; }
inline bool __any(bool v) { return v; }
inline int __ffsll(long long v) { return __builtin_ffsll(v); }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline uint64_t wall_clock64() { return 0; }
inline float __uint_as_float(unsigned v) { return __builtin_bit_cast(float, v); }
inline unsigned __float_as_uint(float v) { return __builtin_bit_cast(unsigned, v); }
inline int __float_as_int(float v) { return __builtin_bit_cast(int, v); }
inline float __int_as_float(int v) { return __builtin_bit_cast(float, v); }
inline unsigned __umulhi(unsigned a, unsigned b) { return (unsigned)(((uint64_t)a * b) >> 32); }
template <typename T, typename U>
T atomicAdd(T* p, U v) {
  const T o = *p;
  *p = (T)(o + v);
  return o;
}
template <typename T, typename U>
T atomicExch(T* p, U v) {
  const T o = *p;
  *p = (T)v;
  return o;
}
template <typename T, typename U>
T atomicMax(T* p, U v) {
  const T o = *p;
  *p = std::max<T>(o, (T)v);
  return o;
}
// uses every operand, so that no load is dropped as dead
template <typename A, typename B, typename C>
C shim_mfma(A a, B b, C c) {
  if constexpr (std::is_arithmetic_v<A>) c += (C)(a * b);
  else c += (float)a[0] * (float)b[0] + (float)a[1] * (float)b[1] + (float)a[2] * (float)b[2] + (float)a[3] * (float)b[3];
  return c;
}
#define __hip_atomic_load(p, ...) (*(p))
#define __hip_atomic_store(p, v, ...) (void)(*(p) = (v))
#define __builtin_amdgcn_fence(...) (void)0
#define __builtin_amdgcn_s_sleep(...) (void)0
#define __builtin_amdgcn_s_waitcnt(...) (void)0
#define __builtin_amdgcn_wave_barrier() (void)0
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_rsq(v) (1.0 / std::sqrt(v))
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, ...) shim_mfma((a), (b), (c))
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, ...) shim_mfma((a), (b), (c))
#define __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, ...) shim_mfma((a), (b), (c))
#define __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, ...) shim_mfma((a), (b), (c))
// the DPP intrinsic is declared by its LLVM name, which no other target has
#define __asm(name)
extern "C" inline double eodabe_dpp_f64(double, double v, int, int, int, bool) { return v; }
