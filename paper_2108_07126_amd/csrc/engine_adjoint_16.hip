// The adjoint kernel of one-wave teams, 16-wide.
#include "adjoint_kernel.h"

namespace pm {

hipError_t launch_adjoint_wave16(const GradParams& a, hipStream_t stream) { return pick_wave16<AdjointRun>(a.p, a, stream); }

}  // namespace pm
