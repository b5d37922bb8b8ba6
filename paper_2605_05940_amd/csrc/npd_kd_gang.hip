// Row-gang KD kernels (npd_kd_gang.hpp): which calls they take, the scratch record they need, and the launch.
#include <atomic>

#include "npd_kd_gang_launch.hpp"

namespace npd {

static std::atomic<int> g_spin_limit{kGangSpinLimitDefault};

int set_gang_spin_limit(int polls) {
  return g_spin_limit.exchange(polls > 0 ? polls : kGangSpinLimitDefault, std::memory_order_relaxed);
}

int gang_spin_limit() { return g_spin_limit.load(std::memory_order_relaxed); }

constexpr int kGangK = 10;      // 128-bit groups per thread and tensor: 80 of a thread's 128 registers hold its slice
constexpr int kGangTopkK = 10;  // top-k teacher: groups per thread of the student row alone
constexpr int kGangSkewK = 6;   // skew forms: the slice is kept as two fp32 values per element from sweep 1 on
constexpr int kGangSkewLongK = 7;  // the same with two of the groups in LDS, see skew_long_slices

static int gang_k(int teacher_kind, int divergence) {
  if (teacher_kind == kTopk) return kGangTopkK;
  return divergence == kSkewKl || divergence == kSkewReverseKl ? kGangSkewK : kGangK;
}

// Slices per row.  A workgroup holds up to k * 256 groups; slices are sized to 8 groups less, because boundaries are moved
// by up to 7 groups so that they are 128-byte boundaries of memory (see launch_kd_gang).
// `on_lines`: every row of the launch begins on a 128-byte boundary, no boundary is ever moved and a slice may be as
// long as a workgroup holds (V = 102,400: 5 full slices instead of 6).
static int gang_slices(int nvec, int k, bool on_lines) {
  const int cap = k * kGangThreads - 8;
  return on_lines ? (nvec + cap + 7) / (cap + 8) : (nvec + cap - 1) / cap;
}
// Rows of less than one and a half slices stay with one workgroup per row (1 is returned): two half-filled slices
// cost more in exchanges than the access order gains (dense teacher, % of the HBM peak, row gangs / one workgroup per
// row: V = 20,480 50 / 72, 24,576 67 / 74, 32,000 73 / 69, 50,304 77 / 69, 100,352 81 / 67).
static int gang_size(int nvec, int k, bool on_lines) {
  const int cap = k * kGangThreads - 8;
  return 2 * nvec < 3 * cap ? 1 : gang_slices(nvec, k, on_lines);
}
static bool rows_on_lines(const KdArgs& a) {
  return a.g != nullptr && (reinterpret_cast<uintptr_t>(a.g) & 127u) == 0 && a.s_stride % 64 == 0;
}

// Gradient calls with a dense teacher (any divergence) or a top-k teacher (forward KL), rows that span at least two
// slices, with or without the CE term of the composite loss at any temperature.
bool gang_path_applies(const KdArgs& a, int teacher_kind, bool want_grad) {
  if ((teacher_kind != kDense && teacher_kind != kTopk) || !want_grad) return false;
  if (a.divergence != kForwardKl && teacher_kind != kDense) return false;
  const int g = gang_size(a.nvec_s, gang_k(teacher_kind, a.divergence), rows_on_lines(a));
  if (g < 2 || g > kGangMax) return false;
  return a.T * (int64_t)g <= 0x7fffffffLL;  // one workgroup per slice, 1-D grid
}

static size_t record_bytes(int64_t T, int g, int words_per_slice) {
  return ((size_t)T * g * words_per_slice + kGangTailWords) * sizeof(uint32_t);
}
size_t gang_workspace_bytes(int64_t T, int32_t V, int teacher_kind, int divergence, bool lse1) {
  const int g = gang_size(V / 8, gang_k(teacher_kind, divergence), false);  // (the larger of the two counts)
  if (g < 2 || T * (int64_t)g > 0x7fffffffLL) return 0;
  if (g > kGangMax && gang_size(V / 8, gang_k(teacher_kind, divergence), true) > kGangMax) return 0;
  return record_bytes(T, g, gang_words(lse1 ? 4 : 2));
}

// Runs in front of the launch of a row-gang kernel whose record carries no numbers (KdArgs::tag): clears the scratch record (and the words behind it) to the
// pattern no posted word takes.
__global__ __launch_bounds__(256) void gang_clear_kernel(uint32_t* ws, size_t words) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256) ws[i] = kGangEmpty;
}

hipError_t clear_gang_record(uint32_t* ws, size_t words, hipStream_t stream) {
  const int64_t want = (int64_t)((words + 1023) / 1024);  // four words per thread
  const int64_t grid = want < 8 * (int64_t)compute_units() ? want : 8 * (int64_t)compute_units();
  return launch_kernel(gang_clear_kernel, dim3((unsigned)grid), dim3(256), 0, stream, ws, words);
}

// Shorter slices, for calls whose workspace has room for their record (gang_workspace_preferred(), at most twice the bytes a
// call asks for; what a call runs does not depend on how much more it was given): groups per thread, 0: none.
// A compute unit works through the slices that fall to it; the fullest one has ceil(slices / 256) of them, so slices of
// another length are judged by that number times their length (a ratio below: shorter slices / slices of 10 groups).
//   5  calls of so few rows that all their slices are resident: five workgroups of 256 threads to a compute unit with sums
//      at tau = 1 (up to 84 registers), six without (78).  They wait for the latency of each step of a slice, not for bytes.
//      With sums at tau = 1 up to 1,280 slices, and to 1,400 where the ratio is at most 9 / 10; else up to 1,320, and to 1,400
//      where the ratio is at most 1.
//      Measured (MI355X, all scored, us of a call, 10 groups / 5), slices of five and ratio in brackets:
//        tau = 1          32 rows of 32,000 10.0 / 8.5; 64 of 50,304 11.8 / 10.9, 264 [1,320, .90] 21.7 / 19.7; 184 of 65,536
//                         [1,288, 1.14] 18.1 / 17.2, 188 [1,316, 1.14] 17.9 / 17.4; 86 of 151,936 [1,290, 1.07] 19.9 / 18.4, 93
//                         [1,395, 1.07] 20.9 / 21.8, 128 [1,920] 24.6 / 27.3; 132 of 100,352 [1,320, 1.0] 20.9 / 19.6; 53 of
//                         262,144 [1,378, 1.0] 21.5 / 21.8
//        tau = 2, NLL     320 of 32,000 [1,280, 1.0] 19.6 / 17.9, 330 [1,320, 1.0] 19.7 / 21.3; 272 of 50,304 [1,360, .90] 23.7 /
//                         23.3 (tau = 3 25.9 / 24.1); 188 of 65,536 [1,316, 1.14] 20.3 / 23.4; 88 of 151,936 [1,320, 1.07] 22.0 / 24.1
//        top-k            322 of 32,000 [1,288, 1.0] 12.8 / 12.3, 340 [1,360, 1.0] 12.9 / 12.7; 50 of 262,144 [1,300, 1.0] 13.8 / 13.2
//   7  tau = 1, rows that two slices of 10 groups fill to four fifths and more, or three to two thirds: one more workgroup
//      per compute unit (94 registers), and no register left empty.  10,000 rows of 36,000 379 / 342, top-k (40 entries)
//      281 / 248; of 40,960 395 / 386, 289 / 275 (32,000 308 / 306, 50,304 475 / 474; with sums at tau = 1 the registers
//      do not allow that workgroup: 36,000 tau = 2 with a CE term 382 / 401).  Fewer rows: from 640 on (top-k 1,024), where
//      a row has no more slices of seven groups than of ten, and where the ratio is below 1, or rows are hardly longer than
//      the shortest of these (top-k: where it is at most 15 / 14 and all slices are resident, six to a compute unit).  Time of 10 groups over time of 7: dense 40,000 351 rows .94, 420 1.12, 512 .95, 600
//      .97, 640 1.03, 1,024 1.02; 42,816 351 1.20; 33,000 351 1.07, 512 1.01; top-k 36,000 470 1.05, 560 .86, 768 .78, 1,024 1.06
// (Rows that are not scored are not known here: their slices count like the others'.)
constexpr int kMeasuredCus = 256;
static int fine_groups(int64_t T, int nvec, int teacher_kind, int divergence, bool lse1, bool on_lines) {
  if (divergence != kForwardKl && divergence != kReverseKl) return 0;
  const bool topk = teacher_kind == kTopk;
  auto fullest = [&](int64_t slices) { return (T * slices + kMeasuredCus - 1) / kMeasuredCus; };
  const int64_t gb = gang_slices(nvec, kGangK, on_lines);
  int64_t g = gang_slices(nvec, 5, on_lines);
  int64_t fine = fullest(g) * gb, base = fullest(gb) * g;  // their quotient is the ratio
  if (g <= kGangMax && T * g <= 1400) {
    if (T * g <= 5 * kMeasuredCus) return 5;
    if (lse1 && !topk ? 10 * fine <= 9 * base : T * g <= 1320 || fine <= base) return 5;
  }
  if (lse1 || nvec <= 4080 || nvec > 5352) return 0;
  g = gang_slices(nvec, 7, on_lines);
  fine = fullest(g) * gb;
  base = fullest(gb) * g;
  const bool many = T >= (topk ? 1024 : 640) || g == gb;
  const bool few = topk ? T * g <= 6 * kMeasuredCus && 14 * fine <= 15 * base : fine < base || nvec <= 4200;
  return many || few ? 7 : 0;
}

// (Which sums at tau = 1 a call takes and where its gradient begins is known at its launch; here the largest record counts.)
size_t gang_workspace_preferred(int64_t T, int32_t V, int teacher_kind, int divergence, bool lse1) {
  const size_t least = gang_workspace_bytes(T, V, teacher_kind, divergence, lse1);
  size_t best = least;
  for (int i = 0; least > 0 && i < (lse1 ? 4 : 2); ++i) {
    const bool on_lines = i & 1, sums = i & 2;
    const int k = fine_groups(T, V / 8, teacher_kind, divergence, sums, on_lines);
    const size_t bytes = k > 0 ? record_bytes(T, gang_slices(V / 8, k, on_lines), gang_words(sums ? 4 : 2)) : 0;
    if (bytes > best && bytes <= 2 * least) best = bytes;
  }
  return best;
}

// Skew forms in longer slices (a record of fewer words than the call has asked for): where that makes them fewer, and the
// slices of six groups are more than are resident at once (1,024, and a call leaves out the rows that are not scored); with
// exponentials of their own at tau = 1 always, where six groups spill 13 registers.  Time of 6 groups over time of 7 (MI355X):
// fewer slices 26,624 1.13, 28,672 1.11, 40,960 1.08, 50,304 1.06, 128,256 1.09, 262,144 1.08; as many 22,528 .998, 32,000 .996,
// 18,432 .98; rows of 65,536, six tenths scored: 200 rows .94, 228 .95, 240 1.10, 300 1.16; 330 of 40,960 .89, 366 1.08; nine
// slices against eight, 209 of 106,439 .98; 119 of 50,304 .92, 39 of 151,936 .95; tau = 3 with a CE term 1.07 .. 1.13, 119 rows of 50,304 .993.
static bool skew_long_slices(const KdArgs& a, bool on_lines) {
  const int64_t g = gang_slices(a.nvec_s, kGangSkewK, on_lines), g_long = gang_slices(a.nvec_s, kGangSkewLongK, on_lines);
  if (g_long < 2) return false;
  return l1_mode(a) == kL1Own || (g_long < g && (a.T * g > 4096 || (a.T * g > 1400 && 7 * g_long <= 6 * g)));
}

template <int DIVK>
static hipError_t launch_gang_skew(const KdArgs& a, bool long_slices, hipStream_t stream) {
  if (long_slices) return launch_gang_dense<DIVK, kGangSkewLongK>(a, stream);
  // (rows that are shared have 2,292 groups at least, two long slices: kL1Own never comes here)
  if (l1_mode(a) == kL1Square)
    return launch_gang_kernel(a, gang_words(4), kd_gang_kernel<kGangSkewK, kDense, kL1Square, DIVK>, stream);
  return launch_gang_kernel(a, gang_words(2), kd_gang_kernel<kGangSkewK, kDense, kL1None, DIVK>, stream);
}

hipError_t launch_kd_gang(const KdArgs& a0, int teacher_kind, size_t workspace_bytes, hipStream_t stream) {
  KdArgs a = a0;
  const bool on_lines = rows_on_lines(a);
  const int base = gang_size(a.nvec_s, gang_k(teacher_kind, a.divergence), on_lines);
  a.gang = base;
  const bool skew = a.divergence == kSkewKl || a.divergence == kSkewReverseKl;
  const bool skew_long = skew && skew_long_slices(a, on_lines);
  if (skew_long) a.gang = gang_slices(a.nvec_s, kGangSkewLongK, on_lines);
  int k = fine_groups(a.T, a.nvec_s, teacher_kind, a.divergence, a.need_lse1 != 0, on_lines);
  if (k > 0) {
    const int g = gang_slices(a.nvec_s, k, on_lines);
    const size_t bytes = record_bytes(a.T, g, gang_words(teacher_kind == kTopk || !a.need_lse1 ? 2 : 4));
    const size_t least =
        gang_workspace_bytes(a.T, a.V, teacher_kind, a.divergence, teacher_kind == kDense && a.c != kLog2e);
    if (g >= 2 && bytes <= workspace_bytes && bytes <= 2 * least)
      a.gang = g;
    else
      k = 0;
  }
  // Slices that are one run of groups (`DEALT` in npd_kd_gang.hpp says which are not) are multiples of 8 groups = 128 bytes long,
  // and the kernels move every boundary inside a row, of runs and of pieces, down to the next 128-byte boundary of the gradient
  // row's address (by 0 .. 7 groups: a row whose pitch is not a multiple of 128 bytes begins anywhere): no cache line is then
  // shared by two workgroups of a row -- measured +2.4 points of the HBM
  // peak on 32,768 x 151,936, +2.5 on 262,144 logits in place, +3.6 with a top-k teacher; a row pitch of 16 bytes more than
  // 151,936 logits: +4.
  a.gang_groups = ((a.nvec_s + a.gang - 1) / a.gang + 7) / 8 * 8;
  a.spin_limit = gang_spin_limit();
  if (k > 0) return launch_gang_fine(a, k, teacher_kind, stream);
  if (teacher_kind == kTopk) return launch_gang_topk<kGangTopkK>(a, stream);
  switch (a.divergence) {
    case kReverseKl: return launch_gang_dense<kReverseKl, kGangK>(a, stream);
    case kSkewKl: return launch_gang_skew<kSkewKl>(a, skew_long, stream);
    case kSkewReverseKl: return launch_gang_skew<kSkewReverseKl>(a, skew_long, stream);
    default: return launch_gang_dense<kForwardKl, kGangK>(a, stream);
  }
}

}  // namespace npd
