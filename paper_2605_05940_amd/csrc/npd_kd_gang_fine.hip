// Row-gang kernels with shorter slices; which calls: fine_groups in npd_kd_gang.hip.
#include "npd_kd_gang_launch.hpp"

namespace npd {

hipError_t launch_gang_fine(const KdArgs& a, int k, int teacher_kind, hipStream_t stream) {
  if (k == 7) {  // no sums at tau = 1
    if (teacher_kind == kTopk) return launch_gang_topk_sums<7, kL1None>(a, stream);
    if (a.divergence == kReverseKl)
      return launch_gang_kernel(a, gang_words(2), kd_gang_kernel<7, kDense, kL1None, kReverseKl>, stream);
    return launch_gang_kernel(a, gang_words(2), kd_gang_kernel<7, kDense, kL1None, kForwardKl>, stream);
  }
  if (teacher_kind == kTopk) return launch_gang_topk<5>(a, stream);
  if (a.divergence == kReverseKl) return launch_gang_dense<kReverseKl, 5>(a, stream);
  return launch_gang_dense<kForwardKl, 5>(a, stream);
}

}  // namespace npd
