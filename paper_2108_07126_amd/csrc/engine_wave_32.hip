// One-wave teams, 32-wide (dimensions 17..32), Taylor series.
#include "wave_kernel.h"

namespace pm {
namespace {

template <int EXPO>
hipError_t launch_k(const PropParams& p, int nb, hipStream_t stream) {
    if (wave_lds_bytes<2>(nb, true) > 160 * 1024) return launch_wave_one<Wide<2, 8>, EXPO, false, false>(p, stream);
    if (p.du <= 24) return launch_wave_one<Wide<2, 6>, EXPO, false, true>(p, stream);
    return p.du <= 28 ? launch_wave_one<Wide<2, 7>, EXPO, false, true>(p, stream)
                      : launch_wave_one<Wide<2, 8>, EXPO, false, true>(p, stream);
}

}  // namespace

// A block keeps up to eight basis matrices in LDS (16 KiB each).  Fourth
// order with three controls has ten: there the exponent is formed on
// {H0, H_k} with one commutator by product.
hipError_t launch_wave32(const PropParams& p, hipStream_t stream) {
    if (p.order == 4 && wave_lds_bytes<2>(p.M, true) > 160 * 1024) return launch_k<EXPO_COMM>(p, p.K + 1, stream);
    return launch_k<EXPO_BASIS>(p, p.M, stream);
}

}  // namespace pm
