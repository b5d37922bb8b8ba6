// Rows that fit one workgroup: which calls, and the kernels without a dense teacher.
#include "npd_kd_solo.hpp"

namespace npd {

// Every call with whole 128-bit groups whose row fits, forward-only calls with the forward KL or without a teacher --
// except where the row-resident kernel with 256 threads (npd_kd_cached.hpp) is a little faster: 16-byte aligned rows
// whose gradient needs no sum at tau = 1, of more than 2,048 groups (forward KL) or 1,536 groups (reverse KL).
// Measured (MI355X, 65,536 rows or what 1e9 logits give, all scored, % of 8 TB/s, the kernel that ran such a row before /
// this one; in parentheses what was left to the other kernel for it):
//   dense, forward KL  V = 1,024 41 / 61, 2,048 51 / 72, 4,096 41 / 77, 8,192 59 / 78, 12,288 69 / 73 (18,432 74 / 75,
//                      24,576 75 / 72);  at tau = 2 with CE 2,048 46 / 70, 8,192 44 / 68, 16,384 49 / 71, 24,576 51 / 61
//   reverse KL         2,048 53 / 79, 8,192 60 / 79, 12,288 69 / 75 (16,384 74 / 70)
//   skew KL            2,048 36 / 79, 8,192 39 / 74, 12,288 43 / 75, 16,384 45 / 67
//   top-k (64), tau 2  2,048 34 / 54, 4,096 35 / 53, 8,192 43 / 62, 16,384 56 / 62, 24,576 59 / 67
//   NLL alone          2,048 72 / 82, 4,096 39 / 84, 8,192 59 / 87, 16,384 88 / 89
// Short rows used to stream twice; a row that lives in registers is read once, and 5 .. 8 waves per SIMD hide its
// reductions.
// What stays with the kernels that ran it before, with both sides (us, that kernel / this one), unless rows are so few
// that each has a compute unit, or a good part of one, to itself (32 rows of 24,576: no teacher 5.5 / 4.9, tau = 3
// 13.4 / 11.2, k = 20 8.6 / 7.1):
//   no teacher, more than 2,048 groups      V = 20,480 1,500 rows 12.1 / 12.9, 20,000 122 / 132; 30,000 512 rows 6.8 / 7.5
//   a sum at tau = 1 without a CE term, 16-byte aligned rows that fill less than 0.72 (tau = 2; else 0.81) of 512 threads
//                                           V = 20,488 4,096 rows tau = 2 104 / 110, tau = 3 104 / 118; 24,576 tau = 3 121 / 129
//                                           (from 2,048 rows and 1,024 rows on; 22,000 640 rows tau = 2 25.4 / 23.5)
//   top-k teacher with up to 32 entries, no sum at tau = 1, aligned rows of 2,561 .. 3,328 groups
//                                           V = 24,576 k = 20 1,024 rows 17.4 / 18.2, 1,500 26.4 / 29.7
//   top-k teacher, forward only, 33 .. 192 entries, aligned rows of 225 .. 512 groups, 48 MB of them and more (a row's
//   record is gathered before its logits have arrived)
//                                           V = 2,048 k = 64 32,768 rows 36.8 / 41.1; 3,072 k = 160 8,192 rows 19.8 / 20.7
constexpr int kSoloForwardGroups = 256 * 8, kSoloReverseGroups = 256 * 6;
constexpr int kFewRows = 256;
static bool solo_dense_applies(const KdArgs& a, bool want_grad) {
  const int n = a.nvec_s;
  if (!want_grad) return a.divergence == kForwardKl && n <= kSoloGroups;
  if (a.divergence != kForwardKl && a.divergence != kReverseKl) return n <= kSoloSkewGroups;
  if (a.ragged || (a.need_lse1 && a.cscale != 0.0f)) return n <= kSoloGroups;
  if (a.need_lse1)
    return n <= kSoloGroups && (n <= 256 * 10 || n >= (l1_mode(a) == kL1Square ? 2944 : 3328) || a.T < (l1_mode(a) == kL1Square ? 8 : 4) * kFewRows);
  return n <= (a.divergence == kForwardKl ? kSoloForwardGroups : kSoloReverseGroups);
}
static bool solo_topk_applies(const KdArgs& a, bool want_grad) {
  const int n = a.nvec_s;
  if (n > kSoloGroups) return false;
  if (a.ragged) return true;
  if (want_grad) return n <= 256 * 10 || n > 256 * 13 || a.need_lse1 || a.k > 32 || a.T <= kFewRows;
  return !(n > 224 && n <= 512 && a.k > 32 && a.k <= 192 && a.T * (int64_t)a.V >= 24000000);
}
bool solo_path_applies(const KdArgs& a, int teacher_kind, bool want_grad) {
  if (a.nvec_s == 0) return false;
  if (teacher_kind == kNone) return a.nvec_s <= (a.T <= kFewRows ? kSoloGroups : kSoloForwardGroups);
  return teacher_kind == kTopk ? solo_topk_applies(a, want_grad) : solo_dense_applies(a, want_grad);
}

hipError_t launch_kd_solo(const KdArgs& a, int teacher_kind, bool want_grad, hipStream_t stream) {
  if (teacher_kind != kDense)
    return want_grad && teacher_kind == kTopk ? launch_solo_student<true>(a, stream) : launch_solo_student<false>(a, stream);
  if (!want_grad) return launch_solo_forward_only(a, stream);
  if (a.divergence == kForwardKl) return launch_solo_forward(a, stream);
  if (a.divergence == kReverseKl) return launch_solo_reverse(a, stream);
  return launch_solo_skew(a, stream);
}

}  // namespace npd
