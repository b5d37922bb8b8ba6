// Rows that fit one workgroup: dense teacher, forward KL with gradient.
#include "npd_kd_solo.hpp"

namespace npd {

hipError_t launch_solo_forward(const KdArgs& a, hipStream_t stream) { return launch_solo_two_sweeps<kForwardKl, true>(a, stream); }

}  // namespace npd
