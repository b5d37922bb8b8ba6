// Rows that fit one workgroup: dense teacher, reverse KL with gradient.
#include "npd_kd_solo.hpp"

namespace npd {

hipError_t launch_solo_reverse(const KdArgs& a, hipStream_t stream) { return launch_solo_two_sweeps<kReverseKl, true>(a, stream); }

}  // namespace npd
