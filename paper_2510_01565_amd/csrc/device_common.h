// Device helpers for gfx950: bf16 storage conversions, wave64 reductions,
// activations, and the numbering of blocks.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "dit_internal.h"

namespace dit {

// Compile-time loop: f(std::integral_constant<int, 0>) ... f(<N-1>).  Register
// arrays indexed by its counter never become dynamically indexed (which would
// move them to scratch memory).
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

typedef uint16_t bf16_t;  // raw bfloat16 storage
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(bf16_t u) { return __uint_as_float(((uint32_t)u) << 16); }

// fp32 -> bf16, round to nearest even (hardware conversion on gfx950)
__device__ __forceinline__ bf16_t f2bf(float f) {
  __bf16 b = (__bf16)f;
  return __builtin_bit_cast(bf16_t, b);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
}

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return bf2f(v); }

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return f2bf(v); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// GELU, tanh form: 0.5 x (1 + tanh(u)) = x * sigmoid(2u), u = sqrt(2/pi) (x + 0.044715 x^3).
// exp2 and the reciprocal are single transcendental-unit instructions (about
// 1 ulp each); for very negative x the exponential overflows to +inf and the
// result is -0.
__device__ __forceinline__ float gelu_tanh(float x) {
  const float k = -2.0f * 0.7978845608028654f * 1.4426950408889634f;  // -2 sqrt(2/pi) log2(e)
  const float t = k * x * (1.0f + 0.044715f * x * x);
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

__device__ __forceinline__ float silu(float x) { return x / (1.0f + __expf(-x)); }

// 16 consecutive values as bf16, with two 16-byte stores.
__device__ __forceinline__ void store16(bf16_t* dst, const float* v) {
  uint4 a, b;
  a.x = pack_bf16x2(v[0], v[1]);
  a.y = pack_bf16x2(v[2], v[3]);
  a.z = pack_bf16x2(v[4], v[5]);
  a.w = pack_bf16x2(v[6], v[7]);
  b.x = pack_bf16x2(v[8], v[9]);
  b.y = pack_bf16x2(v[10], v[11]);
  b.z = pack_bf16x2(v[12], v[13]);
  b.w = pack_bf16x2(v[14], v[15]);
  ((uint4*)dst)[0] = a;
  ((uint4*)dst)[1] = b;
}

// A launch holds fewer than 2^32 threads along x (past that the runtime wraps the
// grid without an error): 256-thread blocks go on along y after every 2^23.
// block_id() numbers them; where blockIdx.y > 0 it may lie past the last block,
// which the kernel ends.
constexpr int kGridRowLog2 = 23;
inline dim3 grid_of(long blocks) {
  return dim3((unsigned)std::min(blocks, 1L << kGridRowLog2), (unsigned)((blocks - 1) >> kGridRowLog2) + 1);
}
__device__ __forceinline__ int block_id() { return (int)(blockIdx.y << kGridRowLog2) + (int)blockIdx.x; }

// Word 3 of a raw buffer resource on gfx9-family targets: 32-bit data format,
// so untyped dword loads are range-checked against num_records and return
// zeros past it.
constexpr int kBufferWord3 = 0x00020000;

// XCD-aware block remap: hardware dispatches block b to XCD b % 8; return an
// index such that every XCD owns one contiguous range of indices.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
  const int per = nblocks / 8, rem = nblocks % 8;
  const int xcd = bid % 8, idx = bid / 8;
  return (xcd < rem) ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

}  // namespace dit
