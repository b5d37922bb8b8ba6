// Row-resident KD kernels, forward KL with gradient, 256 threads per workgroup (see forward_grad_shape for the rows).
#include "npd_kd_cached.hpp"

namespace npd {

// Rows of up to 4,096 groups live in one workgroup's registers where the call wants a sum at tau = 1 or has a top-k teacher
// (npd_kd_solo.hip), except some of 2,561 .. 3,328 groups: 11 .. 13 groups per thread.
template <int CS>
static hipError_t launch_dense(const KdArgs& a, hipStream_t stream) {
  constexpr int CSR = kResidentGroups < CS ? kResidentGroups : CS;
  return launch_cached_lse1<CS, CSR, 9, kAhead, kDense, true, kForwardKl, 256, true, CS != 16>(a, stream);
}
template <int CS>
static hipError_t launch_topk(const KdArgs& a, hipStream_t stream) {  // the LDS parks student groups
  return launch_cached_lse1<CS, kResidentGroups, CS - kResidentGroups, 3, kTopk, true, kForwardKl, 256, true, CS == 19>(
      a, stream);
}

hipError_t launch_cached_short_256(const KdArgs& a, int cs, int teacher_kind, hipStream_t stream) {
  if (teacher_kind == kTopk) return cs == 13 ? launch_topk<13>(a, stream) : launch_topk<19>(a, stream);
  if (cs == 13) return launch_dense<13>(a, stream);
  if (cs == 16) return launch_dense<16>(a, stream);
  return launch_dense<19>(a, stream);
}

}  // namespace npd
