// Value order of bf16 bit patterns as integers, shared by the top-k kernels.
#pragma once
#include "npd_device.hpp"

namespace npd {

typedef short short2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ short2v as_s2(uint32_t x) { return __builtin_bit_cast(short2v, x); }
__device__ __forceinline__ short2v pk_max(short2v a, short2v b) { return __builtin_elementwise_max(a, b); }
__device__ __forceinline__ short2v pk_min(short2v a, short2v b) { return __builtin_elementwise_min(a, b); }
// bf16 bit patterns (sign-magnitude) -> 16-bit two's complement integers in value order (an involution);
// -0 becomes -1, directly below +0
__device__ __forceinline__ uint32_t pk_ordered(uint32_t x) {
  const uint32_t sign = __builtin_bit_cast(uint32_t, as_s2(x) >> (short)15);
  return x ^ (sign & 0x7fff7fffu);
}
__device__ __forceinline__ int ordered_of(uint32_t b) {  // one pattern
  const int x = (int)(short)(uint16_t)b;
  return x < 0 ? (x ^ 0x7fff) : x;
}
// the 16-bit sort key of an ordered integer (the same keys as key_of: -0 is filed under +0)
__device__ __forceinline__ uint32_t key_of_ordered(int o) {
  const uint32_t key = ((uint32_t)o ^ 0x8000u) & 0xffffu;
  return key == 0x7fffu ? 0x8000u : key;
}
__device__ __forceinline__ float value_of_key(uint32_t key) {
  const uint32_t b = (key & 0x8000u) ? (key & 0x7fffu) : (~key & 0xffffu);
  return __builtin_bit_cast(float, b << 16);
}

}  // namespace npd
