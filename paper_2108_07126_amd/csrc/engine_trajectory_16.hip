// The trajectory kernel of one-wave teams, 16-wide.
#include "adjoint_kernel.h"

namespace pm {

hipError_t launch_trajectory_wave16(const TrajParams& a, hipStream_t stream) { return pick_wave16<TrajRun>(a.p, a, stream); }

}  // namespace pm
