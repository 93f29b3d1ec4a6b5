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

namespace {

template <class S, bool BL>
hipError_t launch_cheb(const PropParams& p, hipStream_t stream) {
    return p.M <= kWaveBasis ? launch_wave_one<S, EXPO_BASIS, true, BL>(p, stream)
                             : launch_wave_one<S, EXPO_COMM, true, BL>(p, stream);
}

}  // namespace

// Two tiles wide LDS holds the matrices put aside and the basis stays in memory,
// and the instances reach as many k-slices as the dimension: 28 levels, 16384
// slices 850 -> 426 us against one instance with every matrix in registers (501
// of them spilled), 32 levels 857 -> 473 us.
hipError_t launch_wave_cheb(int D, const PropParams& p, hipStream_t stream) {
    if (D == 32) {
        if (p.du <= 24) return launch_cheb<Wide<2, 6>, false>(p, stream);
        return p.du <= 28 ? launch_cheb<Wide<2, 7>, false>(p, stream) : launch_cheb<Wide<2, 8>, false>(p, stream);
    }
    return launch_cheb<Wide<1, 4>, true>(p, stream);
}

}  // namespace pm
