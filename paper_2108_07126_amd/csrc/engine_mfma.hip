// MFMA engines: the reduced-precision instances of the propagation kernel, and
// the dispatch over precision, dimension and pairing (FP64 runs on one-wave
// teams up to dimension 32 and on strip teams above).
#include "mfma_kernel.h"

namespace pm {

template <int PMODE>
hipError_t launch_dims(int D, const PropParams& p, hipStream_t stream) {
    switch (D) {
        case 16: return launch_bl<float, 16, kNT16, PMODE>(p, stream);
        case 32: return launch_bl<float, 32, 1, PMODE>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_wave(int D, const PropParams& p, hipStream_t stream);
hipError_t launch_strip(const PropParams& p, hipStream_t stream);
hipError_t launch_panel(int precision, const PropParams& p, hipStream_t stream);
hipError_t launch_mfma_pair(int precision, const PropParams& p, hipStream_t stream);

hipError_t launch_mfma(int D, int precision, const PropParams& p, hipStream_t stream) {
    if (p.pair && D != 16) return hipErrorInvalidValue;
    if (precision == PM_FP64) return D == 64 ? launch_strip(p, stream) : launch_wave(D, p, stream);
    if (p.order == kOrderM6) return hipErrorInvalidValue;
    if (D == 64) return launch_panel(precision, p, stream);
    if (p.pair) return launch_mfma_pair(precision, p, stream);
    switch (precision) {
        case PM_FP32: return launch_dims<0>(D, p, stream);
        case PM_FP32_3M: return launch_dims<1>(D, p, stream);
        case PM_BF16_SPLIT: return launch_dims<2>(D, p, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace pm
