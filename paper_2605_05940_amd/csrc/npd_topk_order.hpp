// Value order of bf16 bit patterns as integers, and the ordering of a candidate list by one wave, shared by the top-k
// kernels.
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


// ---- sorting 64 R words in the registers of one wave, largest first: position lane * R + r ends with the word of that
// rank.  A bitonic network in its mirrored form: every run is descending, so a comparison keeps the larger word on the
// side with the smaller position whatever the run.  Partners in other lanes come through DPP and the row swaps of this
// chip, without LDS.  Instructions: about 100 for 64 words, 170 for 128, 420 for 256, 1,000 for 512, against
// n (n / 4) / 64 * 9 of an all-pairs ranking by one wave (130, 560, 2,300, 9,200).
template <int MASK>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
  if constexpr (MASK == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xb1, 0xf, 0xf, true);        // quad_perm 1,0,3,2
  else if constexpr (MASK == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4e, 0xf, 0xf, true);   // quad_perm 2,3,0,1
  else if constexpr (MASK == 3) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x1b, 0xf, 0xf, true);   // quad_perm 3,2,1,0
  else if constexpr (MASK == 7) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xf, 0xf, true);  // row_half_mirror
  else if constexpr (MASK == 15) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x140, 0xf, 0xf, true); // row_mirror
  else if constexpr (MASK == 8) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xf, 0xf, true);  // row_ror:8
  else if constexpr (MASK == 4) return lane_xor<7>(lane_xor<3>(x));
  else if constexpr (MASK == 16) {
    const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);  // rows (0, 0, 2, 2) and (1, 1, 3, 3) of x
    return (threadIdx.x & 16) ? p[0] : p[1];
  } else if constexpr (MASK == 32) {
    const auto p = __builtin_amdgcn_permlane32_swap(x, x, false, false);  // the lower half twice, the upper half twice
    return (threadIdx.x & 32) ? p[0] : p[1];
  } else if constexpr (MASK == 31)
    return lane_xor<16>(lane_xor<15>(x));
  else
    return lane_xor<32>(lane_xor<31>(x));
}
// compares every word with its partner in lane ^ MASK; MIRROR: with register R - 1 - r there
template <int R, int MASK, bool MIRROR>
__device__ __forceinline__ void sort_lanes(uint32_t (&v)[R], int lane) {
  constexpr int top = MASK >= 32 ? 32 : MASK >= 16 ? 16 : MASK >= 8 ? 8 : MASK >= 4 ? 4 : MASK >= 2 ? 2 : 1;
  uint32_t p[R];
#pragma unroll
  for (int r = 0; r < R; ++r) p[r] = lane_xor<MASK>(v[MIRROR ? R - 1 - r : r]);
  const bool upper = (lane & top) != 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t hi = v[r] > p[r] ? v[r] : p[r], lo = v[r] > p[r] ? p[r] : v[r];
    v[r] = upper ? lo : hi;
  }
}
template <int R, int MASK>
__device__ __forceinline__ void sort_registers(uint32_t (&v)[R]) {  // MASK + 1 a power of two: mirrored; else one bit
  constexpr int top = (MASK & (MASK + 1)) == 0 ? (MASK + 1) / 2 : MASK;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (!(r & top)) {
      const uint32_t a = v[r], b = v[r ^ MASK];
      v[r] = a > b ? a : b;
      v[r ^ MASK] = a > b ? b : a;
    }
  }
}
template <int R>
__device__ __forceinline__ void sort_registers_tail(uint32_t (&v)[R]) {  // strides R / 2 .. 1
  if constexpr (R >= 8) sort_registers<R, 4>(v);
  if constexpr (R >= 4) sort_registers<R, 2>(v);
  if constexpr (R >= 2) sort_registers<R, 1>(v);
}
template <int R>
__device__ __forceinline__ void wave_sort(uint32_t (&v)[R], int lane) {
  static_assert(R == 1 || R == 2 || R == 4 || R == 8, "");
  if constexpr (R >= 2) sort_registers<R, 1>(v);
  if constexpr (R >= 4) {
    sort_registers<R, 3>(v);
    sort_registers<R, 1>(v);
  }
  if constexpr (R >= 8) {
    sort_registers<R, 7>(v);
    sort_registers<R, 2>(v);
    sort_registers<R, 1>(v);
  }
  sort_lanes<R, 1, true>(v, lane);
  sort_registers_tail<R>(v);
  sort_lanes<R, 3, true>(v, lane);
  sort_lanes<R, 1, false>(v, lane);
  sort_registers_tail<R>(v);
  sort_lanes<R, 7, true>(v, lane);
  sort_lanes<R, 2, false>(v, lane);
  sort_lanes<R, 1, false>(v, lane);
  sort_registers_tail<R>(v);
  sort_lanes<R, 15, true>(v, lane);
  sort_lanes<R, 4, false>(v, lane);
  sort_lanes<R, 2, false>(v, lane);
  sort_lanes<R, 1, false>(v, lane);
  sort_registers_tail<R>(v);
  sort_lanes<R, 31, true>(v, lane);
  sort_lanes<R, 8, false>(v, lane);
  sort_lanes<R, 4, false>(v, lane);
  sort_lanes<R, 2, false>(v, lane);
  sort_lanes<R, 1, false>(v, lane);
  sort_registers_tail<R>(v);
  sort_lanes<R, 63, true>(v, lane);
  sort_lanes<R, 16, false>(v, lane);
  sort_lanes<R, 8, false>(v, lane);
  sort_lanes<R, 4, false>(v, lane);
  sort_lanes<R, 2, false>(v, lane);
  sort_lanes<R, 1, false>(v, lane);
  sort_registers_tail<R>(v);
}

// A value that at least m of a wave's N x 64 reach, and at most m + slack or as few as can be: bisection on ballots.  `hi` is
// above every value, at least m values are >= lo.
template <int N>
__device__ __forceinline__ int wave_bound(const int (&x)[N], int m, int slack, int lo, int hi) {
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    int n = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) n += __popcll(__ballot(x[i] >= mid));
    if (n >= m) {
      lo = mid;
      if (n <= m + slack) break;
    } else {
      hi = mid;
    }
  }
  return lo;
}

// inclusive prefix over the lanes of a wave
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // lane 15 of rows 0 and 2 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // lane 31 into rows 2 and 3
  return x;
}

// How one 32-bit word holds a candidate: the key above the smallest key of the list, then the id's complement, so that
// larger words come first (the larger key; among equal keys the smaller id).  (Lists are padded with 0, the word of the
// smallest key with the largest id: a candidate of that word is one of several equal words, and reads the same.)
struct CandWord {
  uint32_t key0;  // smallest key
  int id_bits;
  __device__ __forceinline__ uint32_t make(uint32_t key, uint32_t id) const {
    return ((key - key0) << id_bits) | (((1u << id_bits) - 1u) - id);
  }
  __device__ __forceinline__ uint32_t key(uint32_t w) const { return (w >> id_bits) + key0; }
  __device__ __forceinline__ uint32_t id(uint32_t w) const { return ((1u << id_bits) - 1u) - (w & ((1u << id_bits) - 1u)); }
};

// Orders n <= 64 R candidate words and writes the first k <= n as the row's record.  One wave; `load(i)` gives word i.
template <int R, class Load>
__device__ __forceinline__ void wave_order_and_emit(Load load, int n, int k, const CandWord& c, int log_probs, int32_t* irow,
                                                    float* vrow, int lane) {
  uint32_t v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = r * kWave + lane < n ? load(r * kWave + lane) : 0u;
  wave_sort<R>(v, lane);
  float x[R];
#pragma unroll
  for (int r = 0; r < R; ++r) x[r] = value_of_key(c.key(v[r]));
  float lse = 0.0f;
  if (log_probs) {  // log-softmax over the k selected logits; the first one is the largest
    const float v0 = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x[0])));
    float part = 0.0f;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (lane * R + r < k) part += __expf(x[r] - v0);
    lse = v0 + __logf(wave_sum(part));
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = lane * R + r;
    if (j < k) {
      irow[j] = (int32_t)c.id(v[r]);
      vrow[j] = x[r] - lse;
    }
  }
}
constexpr int kWaveSortMax = 8 * kWave;

// The 32-bit form of a list of 64-bit candidates (key above, the id's complement below) of a row of V logits; id_bits < 0 if
// their keys span too much for one.  One wave; every lane returns with the same.
__device__ __forceinline__ CandWord list_word(const unsigned long long* cand, int n, int V, int lane) {
  uint32_t lo = 0xffffu, hi = 0;
  for (int i = lane; i < n; i += kWave) {
    const uint32_t key = (uint32_t)(cand[i] >> 32);
    lo = lo < key ? lo : key;
    hi = hi > key ? hi : key;
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    const uint32_t l2 = (uint32_t)__shfl_xor((int)lo, off, kWave), h2 = (uint32_t)__shfl_xor((int)hi, off, kWave);
    lo = lo < l2 ? lo : l2;
    hi = hi > h2 ? hi : h2;
  }
  lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
  hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
  const int id_bits = V > 1 ? 32 - __builtin_clz((uint32_t)(V - 1)) : 1;
  return CandWord{lo, ((hi - lo) >> (32 - id_bits)) == 0 ? id_bits : -1};
}

// Leaves between k and `most` of the largest of n <= 64 R distinct words in dst (LDS; may be where `load` reads) and returns
// their number (k <= most < n).  One wave.
template <int R, class Load>
__device__ __forceinline__ int wave_cut(Load load, int n, int k, int most, uint32_t* dst, int lane) {
  uint32_t v[R], hi = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    v[r] = r * kWave + lane < n ? load(r * kWave + lane) : 0u;
    hi = hi > v[r] ? hi : v[r];
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    const uint32_t h2 = (uint32_t)__shfl_xor((int)hi, off, kWave);
    hi = hi > h2 ? hi : h2;
  }
  // Bisection: count(>= lo) > most, count(>= hi) < k.  The words are distinct, so the count falls by one at a time and a cut
  // with k .. most words at or above it lies strictly between (k = 1: or it is hi, the largest word).
  hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
  uint32_t lo = 0, cut = hi;
  while (hi - lo > 1) {
    const uint32_t mid = lo + (hi - lo) / 2;
    int c = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) c += __popcll(__ballot(v[r] >= mid));
    if (c > most) {
      lo = mid;
    } else if (c < k) {
      hi = mid;
    } else {
      cut = mid;
      break;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  int at = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const unsigned long long who = __ballot(v[r] >= cut);
    const int pos = at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
    if (v[r] >= cut && pos < most) dst[pos] = v[r];
    at += __popcll(who);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  return at < most ? at : most;
}

// The same for n <= 1,024 candidates and k <= 512; `spare` (LDS, 512 words; may be where `load` reads) is overwritten.
// Lists of more than 64 R words for the smallest R that leaves room for k words and a third are cut first: a cut takes
// some six counts of the registers, a sort of twice the words more than twice the instructions.
template <class Load>
__device__ __forceinline__ void wave_order_and_emit_any(Load load, int n, int k, const CandWord& c, uint32_t* spare,
                                                        int log_probs, int32_t* irow, float* vrow, int lane) {
  const int room = k + k / 3;
  const int most = room <= kWave ? kWave : room <= 2 * kWave ? 2 * kWave : room <= 4 * kWave ? 4 * kWave : kWaveSortMax;
  auto cut_word = [&](int i) { return spare[i]; };
  if (n <= most) {
    if (n <= kWave)
      wave_order_and_emit<1>(load, n, k, c, log_probs, irow, vrow, lane);
    else if (n <= 2 * kWave)
      wave_order_and_emit<2>(load, n, k, c, log_probs, irow, vrow, lane);
    else if (n <= 4 * kWave)
      wave_order_and_emit<4>(load, n, k, c, log_probs, irow, vrow, lane);
    else
      wave_order_and_emit<8>(load, n, k, c, log_probs, irow, vrow, lane);
    return;
  }
  if (n <= 4 * kWave)
    n = wave_cut<4>(load, n, k, most, spare, lane);
  else if (n <= 8 * kWave)
    n = wave_cut<8>(load, n, k, most, spare, lane);
  else
    n = wave_cut<16>(load, n, k, most, spare, lane);
  if (most == kWave)
    wave_order_and_emit<1>(cut_word, n, k, c, log_probs, irow, vrow, lane);
  else if (most == 2 * kWave)
    wave_order_and_emit<2>(cut_word, n, k, c, log_probs, irow, vrow, lane);
  else if (most == 4 * kWave)
    wave_order_and_emit<4>(cut_word, n, k, c, log_probs, irow, vrow, lane);
  else
    wave_order_and_emit<8>(cut_word, n, k, c, log_probs, irow, vrow, lane);
}

}  // namespace npd
