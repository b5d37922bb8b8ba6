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

// The shapes of the forward and the reverse KL.  Forward-only rows of up to 1,536 groups have one of six groups per thread: the
// instances of eight take 101 .. 107 registers since they unpack with the matrix cores, four waves per SIMD, and those of six
// 85 .. 91, five (MI355X, 16,384 rows, us, eight groups unpacked by shifts, five waves / by the matrix cores / six: 8,500 logits
// 89.2 / 97.7 / 84.4, 10,500 101.6 / 108.5 / 99.1; 12,288 113.8 / 111.5 / 114.0).
template <int DIVK, bool GRAD>
static hipError_t launch_solo_two_sweeps(const KdArgs& a, hipStream_t stream) {
  if (a.nvec_s <= 64 * 2) return launch_solo_dense<64, 2, DIVK, GRAD>(a, stream);
  if (a.nvec_s <= 64 * 4) return launch_solo_dense<64, 4, DIVK, GRAD>(a, stream);
  if (a.nvec_s <= 128 * 4) return launch_solo_dense<128, 4, DIVK, GRAD>(a, stream);
  if (a.nvec_s <= 256 * 4) return launch_solo_dense<256, 4, DIVK, GRAD>(a, stream);
  if constexpr (!GRAD)
    if (a.nvec_s <= 256 * 6) return launch_solo_dense<256, 6, DIVK, GRAD>(a, stream);
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
// The shape follows the number of rows and the length of the record beside the row's: a row's record is gathered by its
// threads one entry after another, so a long one, and a row with no others to hide behind, want more threads than the
// logits need.  Measured (MI355X, us; the kernel that ran such rows before / four rows to a workgroup or as few threads
// as hold the row / this rule):
//   32 rows     k = 64  V = 4,096 6.5 / 7.3 / 4.8, 8,192 6.7 / 7.2 / 5.7;  k = 256  4,096 6.7 / 9.9 / 5.2, 8,192 6.9 / 8.6 / 6.1
//               k = 1,000  4,096 8.3 / 11.3 / 7.2, 8,192 8.7 / 12.9 / 6.5, 16,384 9.8 / 10.5 / 7.8, 20,480 10.3 / 11.2 / 7.9
//   8,192 rows  k = 64  V = 4,096 47.6 / 31.7 / 31.7;  k = 256  4,096 49.8 / 51.8 / 40.3, 8,192 87 / 74 / 64
//               k = 1,000  4,096 72 / 78 / 62, 8,192 146 / 129 / 90, 16,384 274 / 172 / 149
// Rows of more than 2,560 groups: 1,024 threads are faster than 512 where fewer than about two rows wait for a place on
// each compute unit and, with one exponential per logit, where many do (28,000 logits, k = 100: 512 rows 13.2 / 12.9,
// 768 17.6 / 18.4, 1,024 22.7 / 23.6, 1,500 39.2 / 34.7, 20,000 444 / 397).
constexpr int kSoloManyRows = 1024;
template <bool GRAD>
static hipError_t launch_solo_student(const KdArgs& a, hipStream_t stream) {
  const int n = a.nvec_s;
  const bool few = a.T < kSoloManyRows;
  // (four rows of 64 threads share the 64 KB of LDS a workgroup gets unasked: records of up to 512 entries)
  if (n <= 64 * 2 && a.k <= 512) return launch_solo_student_shape<64, 2, GRAD>(a, stream);
  if (n <= 128 * 2) {
    if (few || a.k > 512 || (a.k >= 256 && n > 192)) return launch_solo_student_shape<128, 2, GRAD>(a, stream);
    return launch_solo_student_shape<64, 4, GRAD>(a, stream);
  }
  if (n <= 256 * 4 && (few || a.k > (n <= 384 ? 256 : 128))) {
    if (a.k > (n <= 256 * 2 ? 1024 : 512)) return launch_solo_student_shape<512, 2, GRAD>(a, stream);
    if (n <= 256 * 2) return launch_solo_student_shape<256, 2, GRAD>(a, stream);
    return launch_solo_student_shape<256, 4, GRAD>(a, stream);
  }
  if (n <= 64 * 8) return launch_solo_student_shape<64, 8, GRAD>(a, stream);
  if (n <= 128 * 8) return launch_solo_student_shape<128, 8, GRAD>(a, stream);
  if (n <= 512 * 4) {
    if ((few && a.k > 0) || a.k > 256) return launch_solo_student_shape<512, 4, GRAD>(a, stream);
    return launch_solo_student_shape<256, 8, GRAD>(a, stream);
  }
  if (n <= 256 * 10) {
    if (few && a.k > 256) return launch_solo_student_shape<1024, 4, GRAD>(a, stream);
    return launch_solo_student_shape<256, 10, GRAD>(a, stream);
  }
  if ((a.T < 640 && a.k > 0) || (GRAD && !a.need_lse1 && a.T >= 1280)) return launch_solo_student_shape<1024, 4, GRAD>(a, stream);
  return launch_solo_student_shape<512, 8, GRAD>(a, stream);
}

}  // namespace npd
