// Reduced-precision propagation of dimensions 33..64 on panel teams
// (mfma_panel.h): one block of eight waves per chain.
#include "mfma_panel.h"

namespace pm {
namespace {

template <int PMODE, int RT, bool OUT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) propagate_panel(PropParams p) {
    extern __shared__ char lds[];
    const PLane L = panel_lane();
    const int64_t chain = blockIdx.x;
    const int64_t j0 = min(p.n_slices, chain_first(p, chain));
    const int64_t j1 = min(p.n_slices, chain_first(p, chain + 1));
    Tile<double> Q[2];
    panel_run<PMODE, RT, OUT>(p, j0, j1, lds, L, Q);
    const Strip<4> X = panel_to_strips(Q, lds, L);
    if (L.team != 0) return;
    const SLane S{L.lane, L.g, L.j, L.w};
    if (p.chain_out && chain < p.n_chains) strip_node_store<4>(p.chain_out + chain * (int64_t)kPanelD * kPanelD * 2, X, S);
    Slots sl{{lds, lds + strip_slot_bytes<4>()}, 0};
    int* tick = reinterpret_cast<int*>(lds + kPanelLds - 16);
    if constexpr (RT == 4) strip_tree<4, 16, false>(p, blockIdx.x, X, S, sl, tick);
    else if (p.du > 40) strip_tree<4, 12, false>(p, blockIdx.x, X, S, sl, tick);
    else strip_tree<4, 10, false>(p, blockIdx.x, X, S, sl, tick);
}

template <int PMODE, int RT, bool OUT>
hipError_t launch_panel_rt(const PropParams& p, hipStream_t stream) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)propagate_panel<PMODE, RT, OUT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPanelLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((propagate_panel<PMODE, RT, OUT>), dim3((unsigned)p.n_leaves), dim3(512), kPanelLds, stream, p);
    return hipGetLastError();
}

template <int PMODE>
hipError_t launch_panel_mode(const PropParams& p, hipStream_t stream) {
    if (p.slices_out)
        return p.du <= 48 ? launch_panel_rt<PMODE, 3, true>(p, stream) : launch_panel_rt<PMODE, 4, true>(p, stream);
    return p.du <= 48 ? launch_panel_rt<PMODE, 3, false>(p, stream) : launch_panel_rt<PMODE, 4, false>(p, stream);
}

}  // namespace

hipError_t launch_panel(int precision, const PropParams& p, hipStream_t stream) {
    switch (precision) {
        case PM_FP32: return launch_panel_mode<0>(p, stream);
        case PM_FP32_3M: return launch_panel_mode<1>(p, stream);
        case PM_BF16_SPLIT: return launch_panel_mode<2>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace pm
