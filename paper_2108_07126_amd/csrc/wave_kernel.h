// The propagation kernel of one-wave teams (mfma_wave.h), shared by the units
// that instantiate it.
#pragma once
#include "wave_slices.h"

namespace pm {
namespace {

// What bounds it: issue on the SIMD.  No vector instruction overlaps an FP64 MFMA
// of the same SIMD, not even another wave's (measured), so a slice costs its
// MFMAs (16 levels: 48 of 64 cycles) plus its vector instructions (4 cycles
// each at two waves per SIMD, about 7.5 at one).  Cutting the latter from 331
// to about 220 a slice took 16 levels, 2^17 slices from 302 to 272 us.
// One wave per SIMD at D = 32 (four live matrices of 64 registers, the
// accumulators), two at D = 16 (its serial chains of products and plans leave
// gaps that a second wave fills).
template <class S, int EXPO, bool CH, bool BL>
__global__ void __launch_bounds__(64 * kWaveTeams)
__attribute__((amdgpu_waves_per_eu(S::NT == 1 ? 2 : 1, S::NT == 1 ? 8 : 1))) propagate_wave(PropParams p) {
    static_assert(!S::kPair || (EXPO == EXPO_BASIS && !CH), "pairs: Taylor series on the basis");
    constexpr int D = 16 * S::NT;
    using Node = Wide<S::NT, S::kPair ? 2 : S::KS>;   // what enters the tree
    extern __shared__ double wsm[];
    // LDS: the ticket, then the run's part or, at the end, the handover slots
    WLane L;
    L.lane = threadIdx.x & 63;
    L.g = L.lane >> 4;
    L.j = L.lane & 15;
    const int team = wave_uniform((int)(threadIdx.x >> 6));
    int* tick = reinterpret_cast<int*>(wsm);
    d2_t* slots = reinterpret_cast<d2_t*>(wsm + 2);
    if constexpr (BL) {
        block_copy_to_lds(wsm + 2, p.basis, (EXPO == EXPO_BASIS ? p.M : p.K + 1) * S::NT * S::NT * 512);
        __syncthreads();
    }
    WaveSlices<S, EXPO, BL> sl(p, L, wsm + 2, team);

    const int64_t chain = (int64_t)blockIdx.x * kWaveTeams + team;
    const int64_t j0 = min(p.n_slices, chain_first(p, chain));
    const int64_t j1 = min(p.n_slices, chain_first(p, chain + 1));
    // Pair: the chain's halves [j0, jm) and [jm, j1) advance together
    const int64_t jm = S::kPair ? j0 + (j1 - j0 + 1) / 2 : j1;
    const int64_t steps = jm - j0;
    const double lcth = lane_ctheta_of(p, L.lane);
    // Chebyshev, two tiles wide: LDS for two matrices put aside, X and Q
    constexpr bool kAside = CH && S::NT > 1;
    d2_t* aside = reinterpret_cast<d2_t*>(wsm + 2 + wave_run_bytes<S::NT>(sl.nb, BL) / 8) +
                  team * 2 * mx_aside_entries<S>();
    Mx<S> Q = mx_diagonal<S>(L, 1.0);
    sl.start(j0, jm, jm, j1);
    for (int64_t t = 0; t < steps; ++t) {
        Mx<S> E;
        if constexpr (CH) {
            if constexpr (kAside) mx_put_aside<S>(aside + mx_aside_entries<S>(), Q, L);
            Mx<S> G = sl.exponent(t);
            int m, s;
            plan_cheb_lanes(p, wave_uniform(mx_norm1<S>(G)), L.lane, lcth, m, s);
            m = wave_uniform(m);
            s = wave_uniform(s);
            const double sc = ldexp(1.0, -s);
            mx_each<S>([&](int e) {
                G.re[e] *= sc;
                G.im[e] *= sc;
            });
            E = mx_cheb<S>(G, m, p.ctheta[m], p.cheb_j + kChebSplitOffset + m * 2 * kChebHalf, aside, L);
            if (s > 0) mx_square<S>(E, s, sl.scr, L);
            if constexpr (kAside) mx_take_back<S>(Q, aside + mx_aside_entries<S>(), L);
        } else {
            E = sl.slice(t);
        }
        if (p.slices_out) {
            // exp(-i G) = I + E^H: the lane's column of E is a row of the slice
            const int64_t js = sl.second ? jm + t : j0 + t;
            double* out = reinterpret_cast<double*>(p.slices_out) + js * (int64_t)(p.du * p.du) * 2;
            if (js < (sl.second ? j1 : jm))
                mx_each<S>([&](int e) {
                    const int ro = S::col(L, e), co = S::row(L, e);
                    if (ro < p.du && co < p.du)
                        *reinterpret_cast<d2_t*>(out + (ro * p.du + co) * 2) =
                            d2_t{E.re[e] + (ro == co ? 1.0 : 0.0), -E.im[e]};
                });
        }
        if (S::NT > 1 && t == 0) {
            // (two tiles wide the first product, with the identity, is the length
            // of a short chain's whole series: it is a transposition)
            Q = mx_adjoint<S>(E, sl.scr, L);
            mx_each<S>([&](int e) { Q.re[e] += mx_diag<S>(L, e) ? 1.0 : 0.0; });
        } else {
            Q = mx_apply<S>(E, Q);
        }
    }
    Mx<Node> N;
    if constexpr (S::kPair) {
        // the halves' products, second times first, with the identity past
        // the 8 x 8 block: both go through the scratch tile
        d2_t* b = sl.scr + (L.j >> 3) * 72;
        wave_lds_fence();
        mx_each<S>([&](int e) { b[(L.g + 4 * e) * 9 + (L.j & 7)] = d2_t{Q.re[e], Q.im[e]}; });
        wave_lds_fence();
        Mx<Node> A;
        mx_each<Node>([&](int e) {
            const int ro = L.g + 4 * e;
            const bool in = e < S::kRegs && L.j < 8;
            const double id = ro == L.j ? 1.0 : 0.0;
            const d2_t a = sl.scr[in ? 72 + L.j * 9 + ro : 0], x = sl.scr[in ? ro * 9 + L.j : 0];
            A.re[e] = in ? a.x : id;
            A.im[e] = in ? -a.y : 0.0;
            N.re[e] = in ? x.x : id;
            N.im[e] = in ? x.y : 0.0;
        });
        N = mx_join<Node>(A, N, L);
    } else {
        N = Q;
    }
    if (p.chain_out && chain < p.n_chains) {
        double* o = p.chain_out + chain * (int64_t)D * D * 2;
        if constexpr (S::kPair) {
            // the chain's product, and behind it the first half's (the second
            // half's checkpoint): 8 x 8 each
            d2_t* c = reinterpret_cast<d2_t*>(o);
            mx_each<Node>([&](int e) {
                if (e < 2 && L.j < 8) c[(L.g + 4 * e) * 8 + L.j] = d2_t{N.re[e], N.im[e]};
            });
            mx_each<S>([&](int e) {
                if (L.j < 8) c[64 + (L.g + 4 * e) * 8 + L.j] = d2_t{Q.re[e], Q.im[e]};
            });
        } else {
            mx_node_store<Node>(o, N, L);
        }
    }
    // (mx_combine's first barrier comes after every team's last use of the
    // basis and the scratch tiles)
    const Part<Node> B = mx_combine<Node>(N, team, kWaveTeams, slots, L);
    mx_tree<Node>(p, blockIdx.x, B, team, slots, tick, L);
}

// LDS of a launch: a ticket, then the run's part (with `aside` two matrices more
// per team) or the handover slots of the end, whichever is larger.
template <int NT>
constexpr size_t wave_lds_bytes(int nb, bool bl, bool aside = false) {
    const size_t run = wave_run_bytes<NT>(nb, bl) + (aside ? (size_t)kWaveTeams * 2 * NT * NT * 4096 : 0), end = (size_t)kWaveTeams * mx_slot_entries<Wide<NT, 4>>() * 16;
    return 16 + (run > end ? run : end);
}

template <class S, int EXPO, bool CH, bool BL>
hipError_t launch_wave_one(const PropParams& p, hipStream_t stream) {
    const int nb = EXPO == EXPO_BASIS ? p.M : p.K + 1;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)propagate_wave<S, EXPO, CH, BL>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((propagate_wave<S, EXPO, CH, BL>), dim3((unsigned)p.n_leaves), dim3(64 * kWaveTeams),
                       wave_lds_bytes<S::NT>(nb, BL, CH && S::NT > 1), stream, p);
    return hipGetLastError();
}

}  // namespace
}  // namespace pm
