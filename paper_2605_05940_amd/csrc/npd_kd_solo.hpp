// Rows that fit one workgroup's registers: launch of the SOLO forms of the row-gang kernels (npd_kd_gang.hpp,
// npd_kd_gang_topk.hpp).  A shape is TH threads that own K 128-bit groups each per tensor.
#pragma once
#include "npd_kd_gang.hpp"
#include "npd_kd_gang_topk.hpp"

namespace npd {

template <class Kernel>
static hipError_t launch_solo_kernel(const KdArgs& a, int th, size_t lds_bytes, Kernel kernel, hipStream_t stream) {
  const int64_t rows = solo_rows(th);
  return launch_kernel(kernel, dim3((unsigned)((a.T + rows - 1) / rows)), dim3((unsigned)(th * rows)), lds_bytes, stream,
                       a);
}

// dense teacher
template <int TH, int K, int DIVK, bool GRAD>
static hipError_t launch_solo_dense(const KdArgs& a, hipStream_t stream) {
  auto go = [&](auto l1) {
    return launch_solo_kernel(a, TH, 0, kd_gang_kernel<K, kDense, decltype(l1)::value, DIVK, TH, true, GRAD>, stream);
  };
  switch (l1_mode(a)) {
    case kL1None: return go(std::integral_constant<int, kL1None>{});
    case kL1Square: return go(std::integral_constant<int, kL1Square>{});
    default: return go(std::integral_constant<int, kL1Own>{});
  }
}

// the shapes of the forward and the reverse KL
template <int DIVK, bool GRAD>
static hipError_t launch_solo_two_sweeps(const KdArgs& a, hipStream_t stream) {
  if (a.nvec_s <= 64 * 2) return launch_solo_dense<64, 2, DIVK, GRAD>(a, stream);
  if (a.nvec_s <= 64 * 4) return launch_solo_dense<64, 4, DIVK, GRAD>(a, stream);
  if (a.nvec_s <= 128 * 4) return launch_solo_dense<128, 4, DIVK, GRAD>(a, stream);
  if (a.nvec_s <= 256 * 4) return launch_solo_dense<256, 4, DIVK, GRAD>(a, stream);
  if (a.nvec_s <= 256 * 8) return launch_solo_dense<256, 8, DIVK, GRAD>(a, stream);
  if (a.nvec_s <= 256 * 10) return launch_solo_dense<256, 10, DIVK, GRAD>(a, stream);
  return launch_solo_dense<512, 8, DIVK, GRAD>(a, stream);
}
constexpr int kSoloGroups = 512 * 8;

// of the skew forms, which keep two fp32 values per pair of logits
template <int DIVK>
static hipError_t launch_solo_three_sweeps(const KdArgs& a, hipStream_t stream) {
  if (a.nvec_s <= 64 * 2) return launch_solo_dense<64, 2, DIVK, true>(a, stream);
  if (a.nvec_s <= 64 * 4) return launch_solo_dense<64, 4, DIVK, true>(a, stream);
  if (a.nvec_s <= 128 * 4) return launch_solo_dense<128, 4, DIVK, true>(a, stream);
  if (a.nvec_s <= 256 * 4) return launch_solo_dense<256, 4, DIVK, true>(a, stream);
  if (a.nvec_s <= 256 * 6) return launch_solo_dense<256, 6, DIVK, true>(a, stream);
  return launch_solo_dense<512, 5, DIVK, true>(a, stream);
}
constexpr int kSoloSkewGroups = 512 * 5;

// top-k teacher, or none (forward only, k = 0): the student row alone
template <int TH, int K, bool GRAD>
static hipError_t launch_solo_student_shape(const KdArgs& a, hipStream_t stream) {
  const size_t lds = (size_t)solo_rows(TH) * topk_lds_words(TH, K, a.k, GRAD) * sizeof(uint32_t);
  auto go = [&](auto l1) {
    return launch_solo_kernel(a, TH, lds, kd_gang_topk_kernel<K, decltype(l1)::value, TH, true, GRAD>, stream);
  };
  switch (l1_mode(a)) {
    case kL1None: return go(std::integral_constant<int, kL1None>{});
    case kL1Square: return go(std::integral_constant<int, kL1Square>{});
    default: return go(std::integral_constant<int, kL1Own>{});
  }
}
template <bool GRAD>
static hipError_t launch_solo_student(const KdArgs& a, hipStream_t stream) {
  constexpr int kShortRecord = 512;  // four rows of 64 threads share the 64 KB of LDS a workgroup gets unasked
  if (a.k <= kShortRecord) {
    if (a.nvec_s <= 64 * 2) return launch_solo_student_shape<64, 2, GRAD>(a, stream);
    if (a.nvec_s <= 64 * 4) return launch_solo_student_shape<64, 4, GRAD>(a, stream);
    if (a.nvec_s <= 64 * 8) return launch_solo_student_shape<64, 8, GRAD>(a, stream);
  }
  if (a.nvec_s <= 128 * 8) return launch_solo_student_shape<128, 8, GRAD>(a, stream);
  if (a.nvec_s <= 256 * 8) return launch_solo_student_shape<256, 8, GRAD>(a, stream);
  if (a.nvec_s <= 256 * 10) return launch_solo_student_shape<256, 10, GRAD>(a, stream);
  return launch_solo_student_shape<512, 8, GRAD>(a, stream);
}

}  // namespace npd
