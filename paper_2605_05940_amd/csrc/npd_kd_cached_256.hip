// Row-resident KD kernels, forward KL with gradient, 256 threads per workgroup (see forward_grad_shape for the rows).
#include "npd_kd_cached.hpp"

namespace npd {

template <int CS>
static hipError_t launch_short(const KdArgs& a, hipStream_t stream) {
  constexpr int CSR = kResidentGroups < CS ? kResidentGroups : CS;
  return launch_cached_lse1<CS, CSR, 9, kAhead, kDense, true, kForwardKl, 256, true>(a, stream);
}

hipError_t launch_cached_short_256(const KdArgs& a, int cs, int teacher_kind, hipStream_t stream) {
  if (teacher_kind == kTopk) {
    // rows of more than 4,096 groups (shorter ones fit one workgroup, npd_kd_solo.hip): 17 .. 19 groups per thread; the
    // LDS parks student groups
    constexpr int CS = 19, CSR = kResidentGroups;
    return launch_cached_lse1<CS, CSR, CS - CSR, 3, kTopk, true, kForwardKl, 256, true>(a, stream);
  }
  if (cs == 13) return launch_short<13>(a, stream);
  if (cs == 16) return launch_short<16>(a, stream);
  return launch_short<19>(a, stream);
}

}  // namespace npd
