// Rows that fit one workgroup: dense teacher, skew forms with gradient.
#include "npd_kd_solo.hpp"

namespace npd {

hipError_t launch_solo_skew(const KdArgs& a, hipStream_t stream) {
  return a.divergence == kSkewKl ? launch_solo_three_sweeps<kSkewKl>(a, stream)
                                   : launch_solo_three_sweeps<kSkewReverseKl>(a, stream);
}

}  // namespace npd
