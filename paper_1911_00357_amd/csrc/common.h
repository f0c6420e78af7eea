// Device helpers shared by the gfx950 kernels of the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define DEV __device__ __forceinline__

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint16_t bf16_t;  // storage type of bfloat16 values

constexpr int kWave = 64;

// float -> bfloat16, round to nearest even (NaN kept quiet).
DEV bf16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}
DEV float bf2f(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// Loads of a stored element as float, for float or bfloat16 storage.
DEV float ldf(const float* p) { return *p; }
DEV float ldf(const bf16_t* p) { return bf2f(*p); }

// Sum over T aligned lanes (a power of two), in every lane: the butterfly lane ^
// T/2, ..., lane ^ 1.  From 16 lanes on in vector instructions: half-wave and
// row swaps, then rotations of a row of 16, whose partner holds the same bits
// as that of the xor.  A chain of six shuffles through LDS was the longest
// part of a recurrence step (4 envs, 512 units, backward: 994 -> 695 us for 128
// steps).  All lanes active.
template <int T>
DEV float lane_sum(float v) {
  if constexpr (T < 16) {
#pragma unroll
    for (int o = T / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  } else {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    if constexpr (T >= 64) {
      const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
      v = __uint_as_float(r.x) + __uint_as_float(r.y);
    }
    if constexpr (T >= 32) {
      const u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
      v = __uint_as_float(r.x) + __uint_as_float(r.y);
    }
#define ROR_ADD(n) \
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + (n), 0xf, 0xf, false))
    ROR_ADD(8);
    ROR_ADD(4);
    ROR_ADD(2);
    ROR_ADD(1);
#undef ROR_ADD
  }
  return v;
}
DEV float wave_sum(float v) { return lane_sum<64>(v); }
DEV double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
DEV float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
  return v;
}

DEV float sigmoidf_(float x) { return 1.0f / (1.0f + __expf(-x)); }

// Accurate sigmoid/tanh for the recurrent core (expf, not the fast path).
DEV float sigm(float x) { return 1.0f / (1.0f + expf(-x)); }

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }
