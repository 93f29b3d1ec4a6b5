// The trajectory kernel of one-wave teams, 32-wide.
#include "adjoint_kernel.h"

namespace pm {

hipError_t launch_trajectory_wave32(const TrajParams& a, hipStream_t stream) { return pick_wave32<TrajRun>(a.p, a, stream); }

}  // namespace pm
