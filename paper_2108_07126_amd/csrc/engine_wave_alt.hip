// One-wave teams: the sixth-order scheme and the Chebyshev series.
#include "wave_kernel.h"

namespace pm {

hipError_t launch_wave_m6(int D, const PropParams& p, hipStream_t stream) {
    const bool ch = p.method == PM_EXPM_CHEBYSHEV;
    if (D == 16) {
        if (ch) return launch_wave_one<Wide<1, 4>, EXPO_M6, true, true>(p, stream);
        return p.du <= 8 ? launch_wave_one<Wide<1, 2>, EXPO_M6, false, true>(p, stream)
                         : launch_wave_one<Wide<1, 4>, EXPO_M6, false, true>(p, stream);
    }
    if (ch) return launch_wave_one<Wide<2, 8>, EXPO_M6, true, false>(p, stream);
    if (wave_lds_bytes<2>(p.K + 1, true) > 160 * 1024)
        return launch_wave_one<Wide<2, 8>, EXPO_M6, false, false>(p, stream);
    return launch_wave_one<Wide<2, 8>, EXPO_M6, false, true>(p, stream);
}

hipError_t launch_wave_cheb(int D, const PropParams& p, hipStream_t stream) {
    if (D == 32)
        return p.M <= kWaveBasis ? launch_wave_one<Wide<2, 8>, EXPO_BASIS, true, false>(p, stream)
                                 : launch_wave_one<Wide<2, 8>, EXPO_COMM, true, false>(p, stream);
    return p.M <= kWaveBasis ? launch_wave_one<Wide<1, 4>, EXPO_BASIS, true, true>(p, stream)
                             : launch_wave_one<Wide<1, 4>, EXPO_COMM, true, true>(p, stream);
}

}  // namespace pm
