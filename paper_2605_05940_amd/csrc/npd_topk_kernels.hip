// Teacher-side top-k record (Sec. 3.1, "record only the top-k logits"; Alg. 1, Phase 2): for every scored
// position the k vocabulary ids with the largest teacher logits, largest first, equal logits by increasing id,
// and their values (the logits, or their log-softmax over the k).  Exact selection, integer bookkeeping only.
//
// One workgroup per token row, several per CU so that one row's ordering phase overlaps the others' streaming
// (1024 threads, two per CU; for small k 512 threads, four per CU: npd_topk_kernels_512.hip).  Both kernels derive
// a lower bound L of the k-th largest logit from per-thread maxima and append every element >= L as a 64-bit
// (key, ~id) word to an LDS list.  Up to 1,024 candidates are cut and ordered by one wave in its registers
// (npd_topk_order.hpp); longer lists are cut at the k-th key with a two-level radix count and ordered by rank sort
// (bitonic sort for long tie lists).  Rows where more elements pass the bound
// than the list holds (massive ties, constant rows) and k beyond the workgroup size take an exact slow path: binary
// search of the k-th key by counting passes over the row, then the ties of lowest id are collected in id order with
// block-wide scans.
//
// Rows that fit one workgroup's registers have a kernel of their own for k <= 256 (npd_topk_rows.hip).
//
// teacher_topk_stream_kernel (rows of more than 8,192 elements, at any offset) reads each row from HBM once: the
// 16-byte groups of a row are visited in a strided order, so that the first window of groups a thread loads (12 of
// the 19 groups of a 151,936-entry row with 1024 threads) samples the whole vocabulary range; the bound comes from
// that sample alone (the k-th largest of a subset never exceeds the k-th largest of the row), and the rest of the
// row streams through the same register window, compared as packed 16-bit integers.  teacher_topk_kernel (any
// shape) takes the bound from the whole row and reads it twice.
#define NPD_TOPK_NS topk1024
#define NPD_TOPK_TB 1024
#define NPD_TOPK_CAND kTopkMax  // 4096 candidates = 32 KB of LDS: also what the exact slow path leaves behind for any k
// Measured on MI355X, 32,768 x 151,936, k = 10 / 64 / 256: window 8 with a 4-group sample 1.72 / 2.04 / 2.77 ms,
// 8 with 8 1.62 / 1.80 / 2.48, 12 with 12 1.57 / 1.69 / 2.29 (a larger sample gives a tighter bound, hence fewer
// candidates to cut and order); 12 groups are what fits 64 VGPRs, i.e. two workgroups per CU.
#define NPD_TOPK_WINDOW 12
#define NPD_TOPK_SAMPLE 12
#define NPD_TOPK_ANY_SHAPE 1
#define NPD_TOPK_GROUPS 0
#include "npd_topk_impl.hpp"

namespace npd {

namespace topk512 {
hipError_t launch_stream(const TopkArgs& a, hipStream_t stream);  // npd_topk_kernels_512.hip
}

// Which kernel streams a long row.  Many rows: four 512-thread workgroups per CU (three rows stream while a fourth is in
// its ordering phase) as long as their bound, from a sample of eight groups per thread, lets few enough candidates pass;
// else two of 1024 threads.  Up to 512 rows, which is what two per CU hold: 1024 threads.  Up to a row per CU: 1024 threads
// with the whole CU's registers, up to 20 groups in flight per thread and the bound from all of them.
// Measured (MI355X, all scored, us, 512 threads / two of 1024 / one of 1024 per CU; 151,936 logits):
//   128 rows    k = 10 29.8 / 19.8 / 18.6, 64 33.7 / 23.0 / 20.7, 256 371 / 32.0 / 27.1
//   512 rows    k = 10 39.4 / 33.6 / 41.6, 64 43.4 / 37.8 / 44.5
//   2,048 rows  k = 10 105 / 111 / 149, 64 109 / 119 / 162, 128 139 / 130
// Line between the first two (k times chunks of 512 groups): 2,048 rows of 262,144 k = 64 202 / 196, 4,096 362 / 370;
// 8,192 rows of 50,304 k = 256 203 / 271, 65,536 278 / 291; 2,048 rows of 65,536 k = 256 93 / 81.
constexpr int kSmallK = 256;

hipError_t launch_teacher_topk(int64_t T, int32_t V, int64_t stride, int32_t k, int log_probs, const uint16_t* t,
                               const uint8_t* mask, int32_t* idx, float* val, hipStream_t stream) {
  TopkArgs a;
  a.t = t;
  a.mask = mask;
  a.idx = idx;
  a.val = val;
  a.stride = stride;
  a.T = T;
  a.V = V;
  a.k = k;
  a.nvec = V / 8;  // (a row that begins inside a 16-byte group may have one group less)
  a.log_probs = log_probs;
  if (topk_rows_applies(a)) return launch_topk_rows(a, stream);
  // every thread of a workgroup of 1024 needs a whole group
  const bool aligned = (reinterpret_cast<uintptr_t>(t) & 15u) == 0 && stride % 8 == 0;
  if (a.nvec > 1024 || (aligned && a.nvec == 1024)) {
    if (T <= kTopkFewRows) return topk1024::launch_few(a, stream);
    if (T <= 512 && a.nvec > 6144) return topk1024::launch_stream(a, stream);
    // about twice k / 8 candidates per chunk of 512 groups pass the bound of the 512-thread kernel, whose list holds 2,048
    const int64_t chunks = (a.nvec + 511) / 512;
    if (k <= kSmallK && k * chunks <= 8 * (T < 3072 ? 425 : 700)) return topk512::launch_stream(a, stream);
    return topk1024::launch_stream(a, stream);
  }
  if (!aligned) a.nvec = 0;  // element by element: rows this short fit the caches, and few wait for bytes
  return topk1024::launch_any(a, stream);
}

}  // namespace npd
