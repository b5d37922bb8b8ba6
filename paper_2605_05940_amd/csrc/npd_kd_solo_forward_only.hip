// Rows that fit one workgroup: dense teacher, forward KL, forward only.
#include "npd_kd_solo.hpp"

namespace npd {

hipError_t launch_solo_forward_only(const KdArgs& a, hipStream_t stream) { return launch_solo_two_sweeps<kForwardKl, false>(a, stream); }

}  // namespace npd
