// Adjoint gradient and trajectories on one-wave teams (mfma_wave.h): FP64,
// dimensions up to 32, from the checkpoints of a forward pass.
//
// The adjoint.  With W the loss gradient in the convention dL = Re Tr(W^H dU(T)),
// P_j = U_{j-1} ... U_0 and Omega_j = P_j W^H (U_{N-1} ... U_j):
//     dL = Re sum_j Tr(F_j dG_j),  F_j = L_f(G_j, Omega_j U_j^H),  f(G) = exp(-i G),
// (cyclic trace and Tr(A L_f(G, E)) = Tr(L_f(G, A) E)).  U_j commutes with
// G_j, so by L_f(G, E) = -i int_0^1 e^{-isG} E e^{-i(1-s)G} ds
//     F_j = -i phi(K) Omega_j,  Omega_{j+1} = e^K Omega_j,
//     K(X) = -i [G_j, X],  phi(z) = (e^z - 1) / z,
// and dL/dw_{j,m} = Re Tr(F_j B_m) = Tr(Psi_j B_m) with Psi_j = phi(K) Omega_j
// taken on the anti-Hermitian part (Omega - Omega^H) / (2 i) alone: K keeps it
// Hermitian and the basis is Hermitian.  So both follow from one sequence,
// T_0 = Omega, T_k = K(T_{k-1}) / k:
//     Omega_{j+1} = sum T_k,   Psi_j = sum T_k / (k + 1),
// and with X Hermitian, [G, X] = G X - (G X)^H is one product and an adjoint
// read back from LDS.  U_j itself is never formed.  On the 3-qubit register
// that is 13 products a slice; the (value, derivative) series it replaces took
// 26 (8 for the recursion, 18 for the derivative), on two waves.
// ||K|| <= 2 ||G||_2 picks the number of terms.  Past z = 2 the terms grow
// before they fall: there phi and e are taken at K / 2^s and doubled,
// phi(2 K) = (phi(K) + e^K phi(K)) / 2, e^K X = V X V^H with V = exp(-i G / 2^s).
#pragma once
#include "wave_slices.h"

namespace pm {
namespace {

// LDS: the run's part, and where both fit (D = 16) the handover slots behind
// it, otherwise over it (the basis is then copied after the checkpoint).
template <int NT>
constexpr size_t adjoint_lds_bytes(int nb, bool bl) {
    const size_t run = wave_run_bytes<NT>(nb, bl), slots = (size_t)kWaveTeams * mx_slot_entries<Wide<NT, 4>>() * 16;
    return NT == 1 ? run + slots : (run > slots ? run : slots);
}

// The 8 x 8 product at c of a pair forward's chain record, its adjoint's entries.
template <class S>
__device__ __forceinline__ Mx<S> pair_record_adj(const double* c, const WLane& L) {
    Mx<S> A;
    mx_each<S>([&](int e) {
        const d2_t v = reinterpret_cast<const d2_t*>(c)[S::col(L, e) * 8 + S::row(L, e)];
        A.re[e] = v.x;
        A.im[e] = -v.y;
    });
    return A;
}

// P_{j0} = U_{j0-1} ... U_0 for each team's chain (Pair: for both halves),
// from the forward's tree nodes, chain products and first-half products.  The
// leaf's checkpoint is a product of up to seven aligned nodes per tree level
// (base-kFanIn digits of the leaf), a quarter of them per wave; then each
// team multiplies its leaf's earlier chains in.  Every wave of the block calls it.
template <class S>
__device__ __forceinline__ Mx<S> chain_start(const PropParams& p, int64_t leaf, int64_t chain, int team, d2_t* slots,
                                             const WLane& L) {
    using Node = Wide<S::NT, S::kPair ? 2 : S::KS>;
    constexpr int64_t NN = (int64_t)256 * S::NT * S::NT * 2;
    int nlev = 0;
    for (int64_t cnt = p.n_leaves; cnt > 1; cnt = (cnt + kFanIn - 1) / kFanIn) ++nlev;
    int n = 0;
    for (int l = 0; l <= nlev; ++l) n += (int)((leaf >> (kFanInLog2 * l)) & (kFanIn - 1));
    // node number i of the list, earliest leaves (top level) first
    auto node = [&](int i) {
        int l = nlev;
        for (; l > 0; --l) {
            const int d = (int)((leaf >> (kFanInLog2 * l)) & (kFanIn - 1));
            if (i < d) break;
            i -= d;
        }
        int64_t off = 0, cnt = p.n_leaves;
        for (int q = 0; q < l; ++q) {
            off += cnt;
            cnt = (cnt + kFanIn - 1) / kFanIn;
        }
        const int64_t first = (leaf >> (kFanInLog2 * (l + 1))) << kFanInLog2;
        return p.nodes + (off + first + i) * NN;
    };
    Mx<Node> P = mx_diagonal<Node>(L, 1.0);
    const int lo = n * team / kWaveTeams, hi = n * (team + 1) / kWaveTeams;
    if (lo < hi) {
        Mx<Node> X = mx_node_load<Node, false>(node(lo), L), A;
        P = X;
        if (lo + 1 < hi) A = mx_node_load<Node, true>(node(lo + 1), L);
        for (int i = lo + 1; i < hi; ++i) {
            const Mx<Node> cur = A;
            if (i + 1 < hi) A = mx_node_load<Node, true>(node(i + 1), L);
            P = mx_join<Node>(cur, P, L);
        }
    }
    const Part<Node> B = mx_combine<Node>(P, team, kWaveTeams, slots, L);
    __syncthreads();
    constexpr int LD = 16 * S::NT + 1;
    if (B.mine(team))
#pragma unroll
        for (int r = 0; r < 4; ++r) slots[B.row(L, team, r) * LD + B.col(L, team)] = d2_t{B.re[r], B.im[r]};
    __syncthreads();
    Mx<S> R;
    mx_each<S>([&](int e) {
        const d2_t v = slots[S::row(L, e) * LD + S::col(L, e)];
        R.re[e] = v.x;
        R.im[e] = v.y;
    });
    if (chain < p.n_chains) {
        for (int64_t c = leaf * kWaveTeams; c < chain; ++c) {
            const double* rec = p.chain_out + c * NN;
            if constexpr (S::kPair) R = mx_join<S>(pair_record_adj<S>(rec, L), R, L);
            else R = mx_join<S>(mx_node_load<S, true>(rec, L), R, L);
        }
        if constexpr (S::kPair) {
            // the second half starts after the first
            Mx<S> A = pair_record_adj<S>(p.chain_out + chain * NN + 128, L);
            mx_each<S>([&](int e) {
                const bool hi8 = L.j >= 8;
                A.re[e] = hi8 ? A.re[e] : (mx_diag<S>(L, e) ? 1.0 : 0.0);
                A.im[e] = hi8 ? A.im[e] : 0.0;
            });
            R = mx_join<S>(A, R, L);
        }
    }
    return R;
}

// A [rows][cols] complex block (leading dimension ld) as a matrix, zero past it.
template <class S>
__device__ __forceinline__ Mx<S> mx_load_user(const double* a, int rows, int cols, int ld, const WLane& L) {
    Mx<S> m;
    mx_each<S>([&](int e) {
        const int r = S::row(L, e), c = S::col(L, e);
        const bool in = r < rows && c < cols;
        m.re[e] = in ? a[(r * ld + c) * 2 + 0] : 0.0;
        m.im[e] = in ? a[(r * ld + c) * 2 + 1] : 0.0;
    });
    return m;
}

// X - X^H over 2 i: the Hermitian matrix whose i-fold is X's anti-Hermitian part.
template <class S>
__device__ __forceinline__ Mx<S> mx_anti(const Mx<S>& X, d2_t* scr, const WLane& L) {
    const Mx<S> A = mx_adjoint<S>(X, scr, L);
    Mx<S> o;
    mx_each<S>([&](int e) {
        o.re[e] = 0.5 * (X.im[e] - A.im[e]);
        o.im[e] = 0.5 * (A.re[e] - X.re[e]);
    });
    return o;
}

// Sum over the lane's group of eight lanes (Pair) or sixteen.
template <bool PAIR>
__device__ __forceinline__ double group_sum(double x) {
    x += dpp_d<0xB1>(x);    // quad_perm 1 0 3 2
    x += dpp_d<0x4E>(x);    // quad_perm 2 3 0 1
    x += dpp_d<0x141>(x);   // row_half_mirror
    if constexpr (!PAIR) x += dpp_d<0x128>(x);   // row_ror 8
    return x;
}

template <class S, int EXPO, bool BL>
__global__ void __launch_bounds__(64 * kWaveTeams)
__attribute__((amdgpu_waves_per_eu(S::NT == 1 ? 2 : 1, S::NT == 1 ? 8 : 1))) adjoint_wave(GradParams gp) {
    const PropParams& p = gp.p;
    extern __shared__ double wsm[];
    WLane L;
    L.lane = threadIdx.x & 63;
    L.g = L.lane >> 4;
    L.j = L.lane & 15;
    const int team = wave_uniform((int)(threadIdx.x >> 6));
    constexpr bool kBehind = S::NT == 1;
    const int nb = EXPO == EXPO_BASIS ? p.M : p.K + 1;
    constexpr int MAT = S::NT * S::NT * 512;
    d2_t* slots = reinterpret_cast<d2_t*>(wsm + (kBehind ? wave_run_bytes<S::NT>(nb, BL) / 8 : 0));
    if constexpr (BL && kBehind) block_copy_to_lds(wsm, p.basis, nb * MAT);
    // unit: part `part` of every chain of the leaf (Pair: of its halves)
    const int64_t leaf = blockIdx.x / gp.split;
    const int64_t unit = (int64_t)blockIdx.x * kWaveTeams + team;
    const int64_t chain = unit / gp.split, part = unit % gp.split;
    Mx<S> P = chain_start<S>(p, leaf, chain, team, slots, L);
    if constexpr (BL && !kBehind) {
        __syncthreads();
        block_copy_to_lds(wsm, p.basis, nb * MAT);
    }
    __syncthreads();
    if (chain >= p.n_chains) return;   // no block-wide barrier follows
    WaveSlices<S, EXPO, BL> sl(p, L, wsm, team);
    const int64_t c0 = chain * p.chunk, c1 = min(p.n_slices, c0 + p.chunk);
    const int64_t cm = S::kPair ? c0 + (c1 - c0 + 1) / 2 : c1;
    const int64_t sub = (cm - c0 + gp.split - 1) / gp.split;
    const int64_t t0 = min(cm - c0, part * sub), t1 = min(cm - c0, t0 + sub);
    if (t0 >= t1) return;
    sl.start(c0, cm, cm, c1);
    // the unit's predecessors in the chain, recomputed
    for (int64_t t = 0; t < t0; ++t) P = mx_apply<S>(sl.slice(t), P);
    // Omega = P Z P^H, Z the anti-Hermitian part of W^H U(T)
    Mx<S> Om;
    {
        const Mx<S> Z = mx_anti<S>(mx_mul<S>(mx_load_user<S>(gp.W, p.du, p.du, p.du, L),
                                             mx_load_user<S>(gp.UT, p.du, p.du, p.du, L)), sl.scr, L);
        const Mx<S> A = mx_adjoint<S>(P, sl.scr, L);
        Om = mx_mul<S>(A, mx_mul<S>(Z, A));
    }
    const double lth = L.lane < kAdjointTerms ? gp.adth[L.lane] : -1.0;
    const double* cb = EXPO == EXPO_BASIS ? sl.bas : p.basis + L.lane;   // the whole basis
    double* red = reinterpret_cast<double*>(sl.scr);
    for (int64_t t = t0; t < t1; ++t) {
        Mx<S> G = sl.exponent(t);
        double z = 2.0 * sl.step_bound();
        unsigned long long ok = __ballot(z <= lth);
        int s = 0;
        if (!ok) {
            z = fmin(z, 2.0 * mx_norm1<S>(G));
            ok = __ballot(z <= lth);
            if (!ok) {
                s = wave_uniform(min(min_squarings(0.5 * z, fmin(p.sth[p.qmax], 1.0)), 62));
                const double sc = ldexp(1.0, -s);
                z *= sc;
                mx_each<S>([&](int e) {
                    G.re[e] *= sc;
                    G.im[e] *= sc;
                });
                ok = __ballot(z <= lth);
            }
        }
        const int terms = ok ? (int)__builtin_ctzll(ok) + 1 : kAdjointTerms;
        Mx<S> T = Om, Psi = Om, On = Om;
        for (int k = 1; k <= terms; ++k) {
            const Mx<S> Y = mx_mul<S>(G, T);
            const Mx<S> A = mx_adjoint<S>(Y, sl.scr, L);
            const double ik = gp.inv[k], ik1 = gp.inv[k + 1];
            mx_each<S>([&](int e) {
                T.re[e] = (Y.im[e] - A.im[e]) * ik;
                T.im[e] = (A.re[e] - Y.re[e]) * ik;
                On.re[e] += T.re[e];
                On.im[e] += T.im[e];
                Psi.re[e] = fma(ik1, T.re[e], Psi.re[e]);
                Psi.im[e] = fma(ik1, T.im[e], Psi.im[e]);
            });
        }
        if (s > 0) {
            // phi at 2^-s doubled s times, then Omega by the slice itself
            auto conj_by = [&](const Mx<S>& E, const Mx<S>& X) {   // V X V^H of a Hermitian X
                return mx_apply<S>(E, mx_adjoint<S>(mx_apply<S>(E, X), sl.scr, L));
            };
            const int sq = plan_scheme(0.5 * z, lane_sth_of(p, L.lane));
            Mx<S> E = mx_expm1<S>(p, G, wave_uniform(sq < 0 ? p.qmax : sq), L);
            for (int q = 0; q < s; ++q) {
                const Mx<S> C = conj_by(E, Psi);
                mx_each<S>([&](int e) {
                    Psi.re[e] = 0.5 * (Psi.re[e] + C.re[e]);
                    Psi.im[e] = 0.5 * (Psi.im[e] + C.im[e]);
                });
                mx_square<S>(E, 1, sl.scr, L);
            }
            On = conj_by(E, Om);
        }
        Om = On;
        // dL/dw_{j,m} = Tr(Psi B_m): per lane its entries' sum, then over the
        // lanes through LDS, four matrices at a time (row q of lanes sums
        // matrix m0 + q, four lanes' values each)
        constexpr int R = S::kPair ? S::KS : 4;
        const int row = L.lane >> 4, l16 = L.lane & 15;
        const int64_t js = S::kPair && l16 >= 8 ? cm + t : c0 + t;
        const bool write = (l16 & (S::kPair ? 7 : 15)) == 0 && js < (S::kPair && l16 >= 8 ? c1 : cm);
        const int slot = S::kPair ? (L.j >> 3) * 32 + 8 * L.g + (L.j & 7) : L.lane;
        for (int m0 = 0; m0 < p.M; m0 += 4) {
            wave_lds_fence();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int m = min(m0 + q, p.M - 1);
                double acc = 0.0;
#pragma unroll
                for (int i = 0; i < S::NT * S::NT; ++i) {
                    const double* b = cb + (int64_t)m * MAT + i * 512;
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        acc = fma(Psi.re[i * 4 + r], b[r * 64], fma(Psi.im[i * 4 + r], b[256 + r * 64], acc));
                }
                red[q * 64 + slot] = acc;
            }
            wave_lds_fence();
            const d2_t a = *reinterpret_cast<const d2_t*>(red + row * 64 + 4 * l16);
            const d2_t b = *reinterpret_cast<const d2_t*>(red + row * 64 + 4 * l16 + 2);
            const double g = group_sum<S::kPair>((a.x + a.y) + (b.x + b.y));
            const int m = m0 + row;
            if (write && m < p.M) {
                if (!gp.grad_direct) gp.gw[js * p.M + m] = g;
                else if (m >= 1) gp.grad_direct[(int64_t)(m - 1) * p.n_samples + js] = p.h * g;
            }
        }
    }
}

// Trajectory: every prefix P_j (applied to a block of states, or to a density
// matrix), j = 0 .. N: each chain (Pair: half) starts from its checkpoint and
// multiplies its recomputed slices in, writing its rows of the output before
// each slice; the run that ends at N also writes j = N.
template <class S, int EXPO, bool BL>
__global__ void __launch_bounds__(64 * kWaveTeams)
__attribute__((amdgpu_waves_per_eu(S::NT == 1 ? 2 : 1, S::NT == 1 ? 8 : 1))) trajectory_wave(TrajParams tp) {
    const PropParams& p = tp.p;
    extern __shared__ double wsm[];
    WLane L;
    L.lane = threadIdx.x & 63;
    L.g = L.lane >> 4;
    L.j = L.lane & 15;
    const int team = wave_uniform((int)(threadIdx.x >> 6));
    constexpr bool kBehind = S::NT == 1;
    const int nb = EXPO == EXPO_BASIS ? p.M : p.K + 1;
    constexpr int MAT = S::NT * S::NT * 512;
    d2_t* slots = reinterpret_cast<d2_t*>(wsm + (kBehind ? wave_run_bytes<S::NT>(nb, BL) / 8 : 0));
    if constexpr (BL && kBehind) block_copy_to_lds(wsm, p.basis, nb * MAT);
    const int64_t chain = (int64_t)blockIdx.x * kWaveTeams + team;
    Mx<S> X = chain_start<S>(p, blockIdx.x, chain, team, slots, L);
    if constexpr (BL && !kBehind) {
        __syncthreads();
        block_copy_to_lds(wsm, p.basis, nb * MAT);
    }
    __syncthreads();
    if (chain >= p.n_chains) return;   // no block-wide barrier follows
    WaveSlices<S, EXPO, BL> sl(p, L, wsm, team);
    const int64_t c0 = chain * p.chunk, c1 = min(p.n_slices, c0 + p.chunk);
    const int64_t cm = S::kPair ? c0 + (c1 - c0 + 1) / 2 : c1;
    sl.start(c0, cm, cm, c1);
    const int du = p.du;
    const int cols = tp.kind == PM_TRAJ_STATES ? tp.n_vec : du;
    const int64_t stride = (int64_t)du * cols * 2;
    if (tp.kind != PM_TRAJ_PROPAGATORS) {
        const Mx<S> A = mx_adjoint<S>(X, sl.scr, L);
        X = mx_mul<S>(A, mx_load_user<S>(tp.x0, du, cols, cols, L));
        // (P rho) P^H = (P (P rho)^H)^H
        if (tp.kind == PM_TRAJ_DENSITY)
            X = mx_adjoint<S>(mx_mul<S>(A, mx_adjoint<S>(X, sl.scr, L)), sl.scr, L);
    }
    // the commutator-free scheme has two exponentials per slice: a slice
    // boundary is every second one
    const int vs = p.order == kOrderCF4 ? 1 : 0;
    auto store = [&](int64_t j) {
        double* o = tp.out + (j >> vs) * stride;
        mx_each<S>([&](int e) {
            const int r = S::row(L, e), c = S::col(L, e);
            if (r < du && c < cols) *reinterpret_cast<d2_t*>(o + (r * cols + c) * 2) = d2_t{X.re[e], X.im[e]};
        });
    };
    for (int64_t t = 0; t < cm - c0; ++t) {
        const int64_t j = sl.second ? cm + t : c0 + t;
        if ((j & vs) == 0 && j < (sl.second ? c1 : cm)) store(j);
        const Mx<S> E = sl.slice(t);
        X = mx_apply<S>(E, X);
        if (tp.kind == PM_TRAJ_DENSITY)
            X = mx_adjoint<S>(mx_apply<S>(E, mx_adjoint<S>(X, sl.scr, L)), sl.scr, L);
    }
    const int64_t end = sl.second ? c1 : cm;
    if (end == p.n_slices && (!sl.second || c1 > cm)) store(end);
}

template <class S, int EXPO, bool BL>
hipError_t launch_adjoint_one(const GradParams& gp, hipStream_t stream) {
    const int nb = EXPO == EXPO_BASIS ? gp.p.M : gp.p.K + 1;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)adjoint_wave<S, EXPO, BL>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((adjoint_wave<S, EXPO, BL>), dim3((unsigned)(gp.p.n_leaves * gp.split)), dim3(64 * kWaveTeams),
                       adjoint_lds_bytes<S::NT>(nb, BL), stream, gp);
    return hipGetLastError();
}

template <class S, int EXPO, bool BL>
hipError_t launch_traj_one(const TrajParams& tp, hipStream_t stream) {
    const int nb = EXPO == EXPO_BASIS ? tp.p.M : tp.p.K + 1;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)trajectory_wave<S, EXPO, BL>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((trajectory_wave<S, EXPO, BL>), dim3((unsigned)tp.p.n_leaves), dim3(64 * kWaveTeams),
                       adjoint_lds_bytes<S::NT>(nb, BL), stream, tp);
    return hipGetLastError();
}

// The instance for a call, by the forward pass's rules (pairs for dimensions
// <= 8 where it kept pairs; the commutator by product where the basis has
// outgrown LDS).  F::run<S, EXPO, BL>(args).
template <class F, class A>
hipError_t pick_wave16(const PropParams& p, const A& a, hipStream_t stream) {
    if (p.pair)
        return p.du <= 4 ? F::template run<Pair<1>, EXPO_BASIS, true>(a, stream)
                         : F::template run<Pair<2>, EXPO_BASIS, true>(a, stream);
    if (p.M > kWaveBasis) return F::template run<Wide<1, 4>, EXPO_COMM, true>(a, stream);
    return p.du <= 12 ? F::template run<Wide<1, 3>, EXPO_BASIS, true>(a, stream)
                      : F::template run<Wide<1, 4>, EXPO_BASIS, true>(a, stream);
}

template <class F, int EXPO, class A>
hipError_t pick_slices(const PropParams& p, const A& a, hipStream_t stream) {
    if (p.du <= 24) return F::template run<Wide<2, 6>, EXPO, true>(a, stream);
    return p.du <= 28 ? F::template run<Wide<2, 7>, EXPO, true>(a, stream)
                      : F::template run<Wide<2, 8>, EXPO, true>(a, stream);
}

template <class F, class A>
hipError_t pick_wave32(const PropParams& p, const A& a, hipStream_t stream) {
    if (adjoint_lds_bytes<2>(p.M, true) <= 160 * 1024 && p.M <= kWaveBasis)
        return pick_slices<F, EXPO_BASIS>(p, a, stream);
    if (p.order != 4) return F::template run<Wide<2, 8>, EXPO_BASIS, false>(a, stream);
    if (adjoint_lds_bytes<2>(p.K + 1, true) <= 160 * 1024)
        return pick_slices<F, EXPO_COMM>(p, a, stream);
    return F::template run<Wide<2, 8>, EXPO_COMM, false>(a, stream);
}

struct AdjointRun {
    template <class S, int EXPO, bool BL>
    static hipError_t run(const GradParams& a, hipStream_t stream) { return launch_adjoint_one<S, EXPO, BL>(a, stream); }
};
struct TrajRun {
    template <class S, int EXPO, bool BL>
    static hipError_t run(const TrajParams& a, hipStream_t stream) { return launch_traj_one<S, EXPO, BL>(a, stream); }
};

}  // namespace
}  // namespace pm
