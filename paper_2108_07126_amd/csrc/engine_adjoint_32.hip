// The adjoint kernel of one-wave teams, 32-wide.
#include "adjoint_kernel.h"

namespace pm {

hipError_t launch_adjoint_wave32(const GradParams& a, hipStream_t stream) { return pick_wave32<AdjointRun>(a.p, a, stream); }

}  // namespace pm
