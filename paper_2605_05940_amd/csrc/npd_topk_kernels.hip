// Teacher-side top-k record (Sec. 3.1, "record only the top-k logits"; Alg. 1, Phase 2): for every scored
// position the k vocabulary ids with the largest teacher logits, largest first, equal logits by increasing id,
// and their values (the logits, or their log-softmax over the k).  Exact selection, integer bookkeeping only.
//
// One workgroup per token row, several per CU so that one row's ordering phase overlaps the others' streaming
// (512 threads, four per CU: npd_topk_kernels_512.hip; or 1024 threads, two per CU or one: see launch_teacher_topk).  Both kernels derive
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
hipError_t launch_same_channel(const TopkArgs& a, hipStream_t stream);
}

// Which kernel streams a long row.  Four 512-thread workgroups per CU (three rows stream while a fourth is in its ordering
// phase) as long as their bound, from a sample of eight groups per thread, lets few enough groups pass, about k / 4 per chunk
// of 512; else two of 1024 threads.  Up to a row per CU the second choice is one workgroup of 1024 threads with the whole
// CU's registers, up to 20 groups in flight per thread and the bound from all of them, if there are more than the others' 12.
// Where memory alone is the limit (small k, many long rows) two workgroups of 1024 threads read a little faster: up to k = 64;
// where that ends lies with the length (8,192 rows, 512 threads / two of 1024: 100,352 logits k = 72 251 / 254, 128 258 / 276;
// 128,256 k = 72 321 / 316, 128 338 / 332; 200,064 k = 72 510 / 492).
// Measured (MI355X, all scored, us, 512 threads / two of 1024 / one of 1024 per CU), k chunks in brackets:
//   8 rows       65,600 k = 128 [2176] 11.7 / 13.3 / 13.3; 128,256 k = 64 [2048] 15.6 / - / 13.5; 262,144 k = 10 [640] 19.4 / 17.5 / 18.1
//   256 rows     100,352 k = 10 [250] 14.4 / 15.1 / 15.6; 151,936 k = 10 [380] 18.1 / 18.5 / 20.8; 65,600 k = 256 [4352] 29.6 / 18.7 / 18.8
//   512 rows     65,600 k = 64 [1088] 15.4 / 19.1; 151,936 k = 64 [2432] 30.1 / 32.2; 50,304 k = 256 [3328] 27.9 / 23.9
//   1,000 rows   50,304 k = 256 [3328] 34.9 / 40.9; 262,144 k = 64 [4096] 122 / 93
//   4,000 rows   65,600 k = 256 [4352] 116 / 145; 151,936 k = 128 [4864] 210 / 197
//   8,192 rows   100,352 k = 10 249 / 241, 64 254 / 249, 128 261 / 276; 65,600 k = 10 161 / 170
//                100,352 k = 10 243 / 237, 128,256 309 / 305, 200,064 490 / 476, 262,144 670 / 648;  5,700 rows of 151,936
//                k = 10 258 / 259, 200,064 342 / 337, 262,144 470 / 461
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
    const int64_t passing = (int64_t)k * ((a.nvec + 511) / 512);
    const bool few = T <= kTopkFewRows, very_few = T <= kTopkFewRows / 2;
    const int64_t most = very_few && a.nvec > 12288 ? 1300 : few ? 2200 : T <= 512 ? 3250 : T < 3072 ? 3400 : 4400;
    const bool memory_bound = k <= 64 && a.nvec > 12288 && T * a.nvec > 100000000;
    const bool same_channel = stride % 262144 == 0 && k <= 40 && T * a.nvec > 90000000;  // (see load_group)
    if (same_channel) return topk512::launch_same_channel(a, stream);
    const bool threads512 = k <= kSmallK && passing <= most && !memory_bound && !(very_few && a.nvec > 20480);
    if (threads512) return topk512::launch_stream(a, stream);
    return few ? topk1024::launch_few(a, stream) : topk1024::launch_stream(a, stream);
  }
  if (!aligned) a.nvec = 0;  // element by element: rows this short fit the caches, and few wait for bytes
  return topk1024::launch_any(a, stream);
}

}  // namespace npd
