// Launch of the row-gang kernels: the clearing launch in front, and the instance a call's sums at tau = 1 ask for.
#pragma once
#include "npd_kd_gang.hpp"
#include "npd_kd_gang_topk.hpp"

namespace npd {

hipError_t clear_gang_record(uint32_t* ws, size_t words, hipStream_t stream);  // npd_kd_gang.hip

template <class Kernel>
static hipError_t launch_gang_kernel(const KdArgs& a, int words_per_slice, Kernel kernel, hipStream_t stream,
                                     size_t lds_bytes = 0) {
  if (a.tag == 0) {
    const hipError_t e = clear_gang_record(a.ws, (size_t)a.T * a.gang * words_per_slice + kGangTailWords, stream);
    if (e != hipSuccess) return e;
  }
  return launch_kernel(kernel, dim3((unsigned)(a.T * a.gang)), dim3(kGangThreads), lds_bytes, stream, a);
}

template <int DIVK, int K>
static hipError_t launch_gang_dense(const KdArgs& a, hipStream_t stream) {
  switch (l1_mode(a)) {
    case kL1None: return launch_gang_kernel(a, gang_words(2), kd_gang_kernel<K, kDense, kL1None, DIVK>, stream);
    case kL1Square: return launch_gang_kernel(a, gang_words(4), kd_gang_kernel<K, kDense, kL1Square, DIVK>, stream);
    default: return launch_gang_kernel(a, gang_words(4), kd_gang_kernel<K, kDense, kL1Own, DIVK>, stream);
  }
}

template <int K, int L1>
static hipError_t launch_gang_topk_sums(const KdArgs& a, hipStream_t stream) {
  const size_t lds = (size_t)topk_lds_words(kGangThreads, K, a.k, true) * sizeof(uint32_t);
  if (a.ragged) return launch_gang_kernel(a, 8, kd_gang_topk_kernel<K, L1, kGangThreads, false, true, true>, stream, lds);
  return launch_gang_kernel(a, 8, kd_gang_topk_kernel<K, L1>, stream, lds);
}
template <int K>
static hipError_t launch_gang_topk(const KdArgs& a, hipStream_t stream) {
  switch (l1_mode(a)) {
    case kL1None: return launch_gang_topk_sums<K, kL1None>(a, stream);
    case kL1Square: return launch_gang_topk_sums<K, kL1Square>(a, stream);
    default: return launch_gang_topk_sums<K, kL1Own>(a, stream);
  }
}

}  // namespace npd
