// FP64 propagation of dimensions 5..32 on one-wave teams: the choice of the
// instance, and the 16-wide ones of the Taylor series.
#include "wave_kernel.h"

namespace pm {

hipError_t launch_wave32(const PropParams& p, hipStream_t stream);
hipError_t launch_wave_m6(int D, const PropParams& p, hipStream_t stream);
hipError_t launch_wave_cheb(int D, const PropParams& p, hipStream_t stream);

namespace {

hipError_t launch_wave16(const PropParams& p, hipStream_t stream) {
    if (p.pair) return launch_wave_one<Pair<2>, EXPO_BASIS, false, true>(p, stream);
    // past that only fourth order with five controls or more (21 matrices):
    // one commutator by product instead of K (K + 1) / 2 more basis matrices (8
    // levels, 20000 slices, five controls: 52 us, in pairs on 21 matrices 77; eight
    // controls: 60 us, one slice at a time on 45 matrices 247)
    if (p.M > kWaveBasis)
        return p.du <= 8 ? launch_wave_one<Wide<1, 2>, EXPO_COMM, false, true>(p, stream)
                         : launch_wave_one<Wide<1, 4>, EXPO_COMM, false, true>(p, stream);
    return p.du <= 12 ? launch_wave_one<Wide<1, 3>, EXPO_BASIS, false, true>(p, stream)
                      : launch_wave_one<Wide<1, 4>, EXPO_BASIS, false, true>(p, stream);
}

}  // namespace

hipError_t launch_wave(int D, const PropParams& p, hipStream_t stream) {
    if (p.order == kOrderM6) return launch_wave_m6(D, p, stream);
    if (p.method == PM_EXPM_CHEBYSHEV) return launch_wave_cheb(D, p, stream);
    return D == 16 ? launch_wave16(p, stream) : launch_wave32(p, stream);
}

}  // namespace pm
