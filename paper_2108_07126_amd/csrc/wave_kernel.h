// The propagation kernel of one-wave teams (mfma_wave.h), shared by the units
// that instantiate it.
#pragma once
#include "mfma_wave.h"

namespace pm {
namespace {

// How a slice's exponent is formed.
//   EXPO_BASIS  G = sum_m w_m B_m on the whole basis (orders 2, 4, CF4)
//   EXPO_COMM   order 4 on {H0, H_k} with one commutator by product:
//               G = S + i (h^2/12) [A1, A3 - A1], S the Simpson mean; taken
//               where the commutator basis has outgrown LDS
//   EXPO_M6     the sixth-order combination of magnus6_exponent
enum { EXPO_BASIS = 0, EXPO_COMM = 1, EXPO_M6 = 2 };

// Weights of EXPO_COMM: lane 16 q + m holds control m - 1's (m = 0: the
// drift's) weight in S (q = 0), A1 (q = 1) and (h^2/12)(A3 - A1) (q = 2).
__device__ __forceinline__ WeightRecipe comm_recipe(const PropParams& p, int lane) {
    WeightRecipe r;
    const int q = lane >> 4, m = lane & 15;
    r.xb = q;
    r.kind = (q > 2 || m > p.K) ? 5 : (m == 0 ? 0 : 7);
    r.xa = r.kind == 7 ? (int64_t)(m - 1) * p.n_samples : 0;
    return r;
}

__device__ __forceinline__ SliceSamples comm_gather(const PropParams& p, const WeightRecipe& r, int64_t j) {
    SliceSamples v{0.0, 0.0, 0.0, 0.0, 0.0};
    if (p.K == 0) return v;
    const double* a = p.samples + r.xa + 2 * j;
    v.x0 = a[0];
    v.x1 = a[1];
    v.x2 = a[2];
    return v;
}

__device__ __forceinline__ double comm_weight(const PropParams& p, const WeightRecipe& r, const SliceSamples& v) {
    const double h = p.h;
    double w = r.xb == 0 ? (h * (1.0 / 6.0)) * (v.x0 + 4.0 * v.x1 + v.x2)
                         : (r.xb == 1 ? v.x0 : (h * h * (1.0 / 12.0)) * (v.x2 - v.x0));
    w = r.kind == 0 ? (r.xb == 0 ? h : (r.xb == 1 ? 1.0 : 0.0)) : w;
    return r.kind == 5 ? 0.0 : w;
}

__device__ __forceinline__ double comm_bound(double w, float beta) {
    const float t = row16_sum_f(fabsf((float)w) * beta);
    const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 0));
    const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 16));
    const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 32));
    return (double)((s + 2.0f * a * d) * (1.0f + 0x1p-16f));
}

// EXPO_BASIS: the weights of kGroup slices at a time.  Row q of 16 lanes (lane
// 16 q + m, m < M <= 16) holds the weights of the group's slice q (PAIR: of slice
// q & 1 of the first (q < 2) or second half), gathered a group ahead.  One row
// sum and one comparison then bound and plan every slice of the group, and
// the expand step reads its weights back from LDS as broadcasts, instead of
// these steps (about 90 vector instructions) and two lane reads per matrix
// in each slice.

// What bounds it: issue on the SIMD.  No vector instruction overlaps an FP64 MFMA
// of the same SIMD, not even another wave's (measured), so a slice costs its
// MFMAs (16 levels: 48 of 64 cycles) plus its vector instructions (4 cycles
// each at two waves per SIMD, about 7.5 at one).  Cutting the latter from 331
// to about 220 a slice took 16 levels, 2^17 slices from 302 to 272 us.
// One wave per SIMD at D = 32 (four live matrices of 64 registers, the
// accumulators), two at D = 16 (its serial chains of products and plans leave
// gaps that a second wave fills).
template <int NT, int KS, int EXPO, bool CH, bool PAIR, bool BL>
__global__ void __launch_bounds__(64 * kWaveTeams)
__attribute__((amdgpu_waves_per_eu(NT == 1 ? 2 : 1, NT == 1 ? 8 : 1))) propagate_wave(PropParams p) {
    static_assert(!PAIR || (NT == 1 && EXPO == EXPO_BASIS && !CH && KS == 4), "slice pairs");
    constexpr int D = 16 * NT;
    constexpr int MAT = NT * NT * 512;   // doubles of a basis matrix
    constexpr bool kRows = EXPO == EXPO_BASIS;
    constexpr int kGroup = PAIR ? 2 : 4;   // steps per group of weights
    extern __shared__ double wsm[];
    // LDS: [the basis] [a scratch tile per team]; the handover slots of the end
    // lie over both
    const int nb = EXPO == EXPO_BASIS ? p.M : p.K + 1;   // basis matrices used
    WLane L;
    L.lane = threadIdx.x & 63;
    L.g = L.lane >> 4;
    L.j = L.lane & 15;
    const int team = wave_uniform((int)(threadIdx.x >> 6));
    int* tick = reinterpret_cast<int*>(wsm);
    d2_t* slots = reinterpret_cast<d2_t*>(wsm + 2);
    d2_t* scr = reinterpret_cast<d2_t*>(wsm + 2 + (BL ? nb * MAT : 0)) + team * kScratchTile;
    // the group's weights (the wave's 64 lanes) behind the scratch tiles
    double* lw = wsm + 2 + (BL ? nb * MAT : 0) + kWaveTeams * kScratchTile * 2 + team * 64;
    double* lb = wsm + 2;
    if constexpr (BL) {
        block_copy_to_lds(lb, p.basis, nb * MAT);
        __syncthreads();
    }
    const double* bas = (BL ? lb : p.basis) + L.lane;

    const int64_t chain = (int64_t)blockIdx.x * kWaveTeams + team;
    const int64_t j0 = min(p.n_slices, chain_first(p, chain));
    const int64_t j1 = min(p.n_slices, chain_first(p, chain + 1));
    // PAIR: halves [j0, jm) and [jm, j1) advance together, the first in the
    // upper-left 8 x 8 block, the second in the lower-right one
    const int64_t jm = PAIR ? j0 + (j1 - j0 + 1) / 2 : j1;
    const int64_t steps = jm - j0;
    const int row = L.lane >> 4, wlane = L.lane & 15;
    const bool bsecond = PAIR && L.j >= 8;   // this lane's column lies in the second block
    // the run whose weights this lane gathers, and its step within a group
    const int64_t wbase = PAIR && row >= 2 ? jm : j0, wend = PAIR && row >= 2 ? j1 : jm;
    const int wstep = kRows ? (PAIR ? (row & 1) : row) : 0;
    const int64_t jlast = p.n_slices > 0 ? p.n_slices - 1 : 0;
    WeightRecipe wr;
    if constexpr (EXPO == EXPO_M6) wr = m6_recipe(p, L.lane);
    else if constexpr (EXPO == EXPO_COMM) wr = comm_recipe(p, L.lane);
    else wr = weight_recipe(p, wlane);
    auto gather = [&](int64_t t) {
        const int64_t j = min(wbase + wstep + t, jlast);
        if constexpr (EXPO == EXPO_M6) return m6_gather(p, wr, j);
        else if constexpr (EXPO == EXPO_COMM) return comm_gather(p, wr, j);
        else return gather_samples(p, wr, j);
    };
    const float beta = wlane < nb ? p.beta[wlane] : 0.0f;
    const double lsth = kRows ? lane_sth_of(p, wlane) : lane_sth_of(p, L.lane);
    const double lcth = lane_ctheta_of(p, L.lane);
    Sq<NT> Q = sq_diagonal<NT>(L, 1.0);
    SliceSamples smp = gather(0);
    double wl = 0.0;
    float bounds = 0.0f;               // of the row's slice
    unsigned long long fits = 0;       // bit 16 q + s: scheme s serves the row's slice
    for (int64_t t = 0; t < steps; ++t) {
        const int tg = kRows ? (int)(t & (kGroup - 1)) : 0;
        if (!kRows || tg == 0) {
            if constexpr (EXPO == EXPO_M6) wl = m6_weight(p, wr, smp);
            else if constexpr (EXPO == EXPO_COMM) wl = comm_weight(p, wr, smp);
            else wl = combine_weight(p, wr, smp);
            // steps past the run (an odd half of a pair, the end of a group)
            if (kRows && wbase + wstep + t >= wend) wl = 0.0;
            smp = gather(t + (kRows ? kGroup : 1));
            if constexpr (kRows) {
                bounds = row16_sum_f(fabsf((float)wl) * beta) * (1.0f + 0x1p-18f);
                fits = __ballot((double)bounds <= lsth);
                wave_lds_fence();
                lw[L.lane] = wl;
                wave_lds_fence();
            }
        }
        Sq<NT> G = sq_diagonal<NT>(L, 0.0);
        auto load = [&](int m, int i, int n, double (&v)[8]) {
            const double* b = bas + m * MAT + (i * NT + n) * 512;
#pragma unroll
            for (int r = 0; r < 8; ++r) v[r] = b[r * 64];
        };
        auto addto = [&](Sq<NT>& A, int i, int n, double w, const double (&v)[8]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                A.t[i][n].re[r] = fma(w, v[r], A.t[i][n].re[r]);
                A.t[i][n].im[r] = fma(w, v[4 + r], A.t[i][n].im[r]);
            }
        };
        double bound = 0.0;
        if constexpr (kRows) {
            // weights of this step: row tg (PAIR: rows tg and 2 + tg, by column)
            const double* w = lw + 16 * tg + (bsecond ? 32 : 0);
            // the entries of four (D = 16) basis matrices are loaded before
            // their FMAs, so the load latencies overlap
            constexpr int B = NT == 1 ? 4 : 1;
            int m = 0;
            for (; m + B <= nb; m += B) {
                double wv[B];
#pragma unroll
                for (int q = 0; q < B; ++q) wv[q] = w[m + q];
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    double x[B][NT][8];
#pragma unroll
                    for (int q = 0; q < B; ++q)
#pragma unroll
                        for (int n = 0; n < NT; ++n) load(m + q, i, n, x[q][n]);
#pragma unroll
                    for (int q = 0; q < B; ++q)
#pragma unroll
                        for (int n = 0; n < NT; ++n) addto(G, i, n, wv[q], x[q][n]);
                }
            }
            for (; m < nb; ++m) {
                double v[8];
                load(m, 0, 0, v);
                addto(G, 0, 0, w[m], v);
            }
        } else {
            Sq<NT> P2 = G, P3 = G;
            for (int m = 0; m < nb; ++m) {
                const double w1 = readlane_d(wl, m), w2 = readlane_d(wl, 16 + m), w3 = readlane_d(wl, 32 + m);
#pragma unroll
                for (int i = 0; i < NT; ++i)
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        double v[8];
                        load(m, i, n, v);
                        addto(G, i, n, w1, v);
                        addto(P2, i, n, w2, v);
                        addto(P3, i, n, w3, v);
                    }
            }
            if constexpr (EXPO == EXPO_COMM) {
                const Sq<NT> K = sq_commutator<NT, KS>(P2, P3, scr, L);
                sq_each<NT>([&](int i, int n, int r) {
                    G.t[i][n].re[r] -= K.t[i][n].im[r];
                    G.t[i][n].im[r] += K.t[i][n].re[r];
                });
                bound = comm_bound(wl, beta);
            } else {
                // R1 = -i[P1, P2], R2 = (i/60)[P1, 2 P3 + R1],
                // G = P1 + P3/12 - (i/240)[-20 P1 - P3 + R1, P2 + R2]; -i K of a
                // commutator K is (K_im, -K_re)
                Sq<NT> K = sq_commutator<NT, KS>(G, P2, scr, L), W, X;
                sq_each<NT>([&](int i, int n, int r) {
                    const double r1r = K.t[i][n].im[r], r1i = -K.t[i][n].re[r];
                    W.t[i][n].re[r] = 2.0 * P3.t[i][n].re[r] + r1r;
                    W.t[i][n].im[r] = 2.0 * P3.t[i][n].im[r] + r1i;
                    X.t[i][n].re[r] = (-20.0 * G.t[i][n].re[r] - P3.t[i][n].re[r]) + r1r;
                    X.t[i][n].im[r] = (-20.0 * G.t[i][n].im[r] - P3.t[i][n].im[r]) + r1i;
                });
                K = sq_commutator<NT, KS>(G, W, scr, L);
                sq_each<NT>([&](int i, int n, int r) {
                    W.t[i][n].re[r] = P2.t[i][n].re[r] - K.t[i][n].im[r] * (1.0 / 60.0);
                    W.t[i][n].im[r] = P2.t[i][n].im[r] + K.t[i][n].re[r] * (1.0 / 60.0);
                });
                K = sq_commutator<NT, KS>(X, W, scr, L);
                sq_each<NT>([&](int i, int n, int r) {
                    G.t[i][n].re[r] =
                        (G.t[i][n].re[r] + P3.t[i][n].re[r] * (1.0 / 12.0)) + K.t[i][n].im[r] * (1.0 / 240.0);
                    G.t[i][n].im[r] =
                        (G.t[i][n].im[r] + P3.t[i][n].im[r] * (1.0 / 12.0)) - K.t[i][n].re[r] * (1.0 / 240.0);
                });
                bound = m6_bound(wl, beta);
            }
        }
        Sq<NT> E;
        int s = 0;
        auto scale = [&]() {
            const double sc = ldexp(1.0, -s);
            sq_each<NT>([&](int i, int n, int r) {
                G.t[i][n].re[r] *= sc;
                G.t[i][n].im[r] *= sc;
            });
        };
        if constexpr (CH) {
            int m;
            plan_cheb_lanes(p, wave_uniform(sq_norm1<NT>(G)), L.lane, lcth, m, s);
            m = wave_uniform(m);
            s = wave_uniform(s);
            scale();
            E = sq_cheb<NT, KS>(G, m, p.ctheta[m], p.cheb_j + kChebSplitOffset + m * 2 * kChebHalf, L);
        } else {
            int q;
            if constexpr (kRows) {
                const unsigned a = (unsigned)(fits >> (16 * tg)) & 0xffffu;
                const unsigned c = PAIR ? (unsigned)(fits >> (32 + 16 * tg)) & 0xffffu : a;
                q = a && c && p.force_s < 0 ? max(__builtin_ctz(a), __builtin_ctz(c)) : -1;
                if (q < 0) {
                    auto of = [&](int r) {
                        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bounds), 16 * r));
                    };
                    bound = PAIR ? fmaxf(of(tg), of(2 + tg)) : of(tg);
                }
            } else {
                q = p.force_s >= 0 ? -1 : plan_scheme(bound, lsth);
            }
            if (q < 0) {
                // squarings: the exponent's own 1-norm may be the smaller bound
                // (terms that cancel)
                plan_scheme_s(p, fmin(bound, sq_norm1<NT>(G)), L.lane, lane_sth_of(p, L.lane), q, s);
                s = wave_uniform(s);
                scale();
            }
            E = sq_expm1<NT, KS, PAIR>(p, G, wave_uniform(q), L);
        }
        if (s > 0) {
            if constexpr (PAIR) pair_mask(E.t[0][0], L.j);
            sq_square<NT, KS>(E, s, scr, L);
        }
        if (p.slices_out) {
            // exp(-i G) = I + E^H: the lane's column of E is a row of the slice
            const int64_t dd = (int64_t)p.du * p.du;
            double* out = reinterpret_cast<double*>(p.slices_out);
            if constexpr (PAIR) {
                const int64_t js = bsecond ? jm + t : j0 + t;
                const int ro = L.j & 7;
                if (ro < p.du && js < (bsecond ? j1 : jm)) {
                    double* o = out + (js * dd + (int64_t)ro * p.du) * 2;
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const int col = L.g + 4 * r;
                        const double re = bsecond ? E.t[0][0].re[r + 2] : E.t[0][0].re[r];
                        const double im = bsecond ? E.t[0][0].im[r + 2] : E.t[0][0].im[r];
                        if (col < p.du) {
                            o[2 * col + 0] = re + (ro == col ? 1.0 : 0.0);
                            o[2 * col + 1] = -im;
                        }
                    }
                }
            } else {
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    const int ro = 16 * n + L.j;
                    if (ro < p.du) {
                        double* o = out + ((j0 + t) * dd + (int64_t)ro * p.du) * 2;
#pragma unroll
                        for (int i = 0; i < NT; ++i)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int col = 16 * i + L.g + 4 * r;
                                if (col < p.du) {
                                    o[2 * col + 0] = E.t[i][n].re[r] + (ro == col ? 1.0 : 0.0);
                                    o[2 * col + 1] = -E.t[i][n].im[r];
                                }
                            }
                    }
                }
            }
        }
        sq_add<NT>(Q, sq_mul<NT, KS, PAIR>(E, Q));
    }
    if constexpr (PAIR) {
        // the halves' products: second times first, in the upper-left block,
        // with the identity elsewhere
        pair_mask(Q.t[0][0], L.j);
        Sq<NT> S, X;
        wave_lds_fence();
#pragma unroll
        for (int r = 0; r < 4; ++r)
            scr[(L.g + 4 * r) * 17 + L.j] = d2_t{Q.t[0][0].re[r], Q.t[0][0].im[r]};
        wave_lds_fence();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ro = L.g + 4 * r;
            const bool in = r < 2 && L.j < 8;
            const double id = ro == L.j ? 1.0 : 0.0;
            const d2_t a = scr[in ? (L.j + 8) * 17 + ro + 8 : 0];   // the second half's adjoint
            S.t[0][0].re[r] = in ? a.x : id;
            S.t[0][0].im[r] = in ? -a.y : 0.0;
            X.t[0][0].re[r] = in ? Q.t[0][0].re[r] : id;
            X.t[0][0].im[r] = in ? Q.t[0][0].im[r] : 0.0;
        }
        Q = sq_mul<NT, KS>(S, X);
    }
    if (p.chain_out && chain < p.n_chains)
        sq_node_store<NT>(p.chain_out + chain * (int64_t)D * D * 2, Q, L);
    // (sq_combine's first barrier comes after every team's last use of the
    // basis and the scratch tiles)
    sq_combine<NT, KS>(Q, team, kWaveTeams, slots, L);
    sq_tree<NT, KS>(p, blockIdx.x, Q, team, slots, tick, L);
}

// LDS of a launch: the basis (BL), a scratch tile and 64 weights per team, or the
// handover slots of the end, whichever is larger, after a 16-byte ticket.
template <int NT>
constexpr size_t wave_lds_bytes(int nb, bool bl) {
    const size_t run = (bl ? (size_t)nb * NT * NT * 4096 : 0) + (size_t)kWaveTeams * (kScratchTile * 16 + 512);
    const size_t end = (size_t)kWaveTeams * sq_slot_entries<NT>() * 16;
    return 16 + (run > end ? run : end);
}

template <int NT, int KS, int EXPO, bool CH, bool PAIR, bool BL>
hipError_t launch_wave_one(const PropParams& p, hipStream_t stream) {
    const int nb = EXPO == EXPO_BASIS ? p.M : p.K + 1;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)propagate_wave<NT, KS, EXPO, CH, PAIR, BL>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((propagate_wave<NT, KS, EXPO, CH, PAIR, BL>), dim3((unsigned)p.n_leaves), dim3(64 * kWaveTeams),
                       wave_lds_bytes<NT>(nb, BL), stream, p);
    return hipGetLastError();
}

}  // namespace
}  // namespace pm
