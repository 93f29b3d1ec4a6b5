// The slices of a one-wave team's run: weights, exponents and plans, shared by
// the propagation, adjoint and trajectory kernels of mfma_wave.h.
#pragma once
#include "mfma_wave.h"

namespace pm {
namespace {

// How a slice's exponent is formed.
//   EXPO_BASIS  G = sum_m w_m B_m on the whole basis (orders 2, 4, CF4),
//               M <= kWaveBasis
//   EXPO_COMM   order 4 on {H0, H_k} with one commutator by product:
//               G = S + i (h^2/12) [A1, A3 - A1], S the Simpson mean; taken
//               where the commutator basis has outgrown LDS
//   EXPO_M6     sixth order: G = P1 + P3/12 - (i/240)[-20 P1 - P3 + R1, P2 + R2],
//               R1 = -i[P1, P2], R2 = (i/60)[P1, 2 P3 + R1] (the scheme of
//               PM_ORDER_MAGNUS6 on Hermitian matrices)
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

__device__ __forceinline__ double comm_bound(double w, double beta) {
    const float t = row16_sum_f(term_bound(w, beta));
    const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 0));
    const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 16));
    const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 32));
    return (double)((s + 2.0f * a * d) * (1.0f + 0x1p-16f));
}

// LDS of a team's block: the basis (BL), then per team a scratch tile and the
// 64 weights of a group.
template <int NT>
constexpr size_t wave_run_bytes(int nb, bool bl) {
    return (bl ? (size_t)nb * NT * NT * 4096 : 0) + (size_t)kWaveTeams * (kScratchTile * 16 + 512);
}

// Consecutive slices first, first + 1, .. of one run (Pair: of two runs).
//
// EXPO_BASIS takes the weights of kGroup slices at a time.  Row q of 16 lanes
// (lane 16 q + m, m < M <= 16) holds the weights of the group's slice q (Pair: of
// slice q & 1 of the first (q < 2) or second run), gathered a group ahead.  One
// row sum and one comparison then bound and plan every slice of the group, and
// the expand step reads its weights back from LDS as broadcasts, instead of
// these steps (about 90 vector instructions) and two lane reads per matrix in
// each slice.
template <class S, int EXPO, bool BL>
struct WaveSlices {
    static constexpr int NT = S::NT;
    static constexpr int MAT = NT * NT * 512;   // doubles of a basis matrix
    static constexpr bool kRows = EXPO == EXPO_BASIS;
    static constexpr int kGroup = S::kPair ? 2 : 4;

    const PropParams& p;
    const WLane& L;
    d2_t* scr;
    double* lw;
    const double* bas;       // Wide: the lane's entries; Pair: the lane's column of the first block
    int nb, wstep;
    bool second;             // Pair: this lane's column lies in the second matrix
    int64_t wbase, wend, jlast;
    WeightRecipe wr;
    double beta, lsth, wl;
    SliceSamples smp;
    float bounds;            // of the row's slice
    double bound;            // of this step's slice (Pair: the larger), once planned
    unsigned long long fits; // bit 16 q + s: scheme s serves the row's slice
    int tg;

    // lds: the block's LDS laid out as wave_run_bytes says, its basis copied.
    __device__ __forceinline__ WaveSlices(const PropParams& p_, const WLane& L_, double* lds, int team)
        : p(p_), L(L_) {
        nb = EXPO == EXPO_BASIS ? p.M : p.K + 1;
        double* rest = lds + (BL ? nb * MAT : 0);
        scr = reinterpret_cast<d2_t*>(rest) + team * kScratchTile;
        lw = rest + kWaveTeams * kScratchTile * 2 + team * 64;
        bas = (BL ? lds : p.basis) + (S::kPair ? 16 * L.g + (L.j & 7) : L.lane);
        second = S::kPair && L.j >= 8;
        const int wlane = L.lane & 15, row = L.lane >> 4;
        wstep = kRows ? (S::kPair ? (row & 1) : row) : 0;
        jlast = p.n_slices > 0 ? p.n_slices - 1 : 0;
        if constexpr (EXPO == EXPO_M6) wr = m6_recipe(p, L.lane);
        else if constexpr (EXPO == EXPO_COMM) wr = comm_recipe(p, L.lane);
        else wr = weight_recipe(p, wlane);
        beta = wlane < nb ? p.beta[wlane] : 0.0;
        // (the commutator's factors share its h^2, so that neither bound leaves FP32)
        if constexpr (EXPO == EXPO_COMM) beta *= row == 1 ? p.h : (row == 2 ? 1.0 / p.h : 1.0);
        lsth = lane_sth_of(p, kRows ? wlane : L.lane);
        wl = 0.0;
        bounds = 0.0f;
        fits = 0;
    }

    // Start (again) at slice a0 of a run that ends at a1 (Pair: and at b0, b1).
    __device__ __forceinline__ void start(int64_t a0, int64_t a1, int64_t b0, int64_t b1) {
        const bool sec = S::kPair && L.lane >= 32;
        wbase = sec ? b0 : a0;
        wend = sec ? b1 : a1;
        smp = gather(0);
    }

    __device__ __forceinline__ SliceSamples gather(int64_t t) const {
        const int64_t j = min(wbase + wstep + t, jlast);
        if constexpr (EXPO == EXPO_M6) return m6_gather(p, wr, j);
        else if constexpr (EXPO == EXPO_COMM) return comm_gather(p, wr, j);
        else return gather_samples(p, wr, j);
    }

    __device__ __forceinline__ void load(int m, int i, int n, double (&v)[2 * (S::kPair ? S::KS : 4)]) const {
        constexpr int R = S::kPair ? S::KS : 4;
        const double* b = bas + m * MAT + (i * NT + n) * 512;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v[r] = b[r * 64];
            v[R + r] = b[256 + r * 64];
        }
    }
    static __device__ __forceinline__ void addto(Mx<S>& A, int i, int n, double w,
                                                 const double (&v)[2 * (S::kPair ? S::KS : 4)]) {
        constexpr int R = S::kPair ? S::KS : 4;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = (i * NT + n) * 4 + r;
            A.re[e] = fma(w, v[r], A.re[e]);
            A.im[e] = fma(w, v[R + r], A.im[e]);
        }
    }

    // The exponent of step t (steps in order from 0 after start()).
    __device__ __forceinline__ Mx<S> exponent(int64_t t) {
        constexpr int R = S::kPair ? S::KS : 4;
        tg = kRows ? (int)(t & (kGroup - 1)) : 0;
        if (!kRows || tg == 0) {
            if constexpr (EXPO == EXPO_M6) wl = m6_weight(p, wr, smp);
            else if constexpr (EXPO == EXPO_COMM) wl = comm_weight(p, wr, smp);
            else wl = combine_weight(p, wr, smp);
            // steps past the run (an odd half of a pair, the end of a group)
            if (kRows && wbase + wstep + t >= wend) wl = 0.0;
            smp = gather(t + (kRows ? kGroup : 1));
            if constexpr (kRows) {
                bounds = row16_sum_f(term_bound(wl, beta)) * (1.0f + 0x1p-18f);
                fits = __ballot((double)bounds <= lsth);
                wave_lds_fence();
                lw[L.lane] = wl;
                wave_lds_fence();
            }
        }
        Mx<S> G;
        mx_each<S>([&](int e) { G.re[e] = G.im[e] = 0.0; });
        if constexpr (kRows) {
            // weights of this step: row tg (Pair: rows tg and 2 + tg, by column)
            const double* w = lw + 16 * tg + (second ? 32 : 0);
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
                    double x[B][NT][2 * R];
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
                double v[2 * R];
                load(m, 0, 0, v);
                addto(G, 0, 0, w[m], v);
            }
        } else {
            Mx<S> P2 = G, P3 = G;
            for (int m = 0; m < nb; ++m) {
                const double w1 = readlane_d(wl, m), w2 = readlane_d(wl, 16 + m), w3 = readlane_d(wl, 32 + m);
#pragma unroll
                for (int i = 0; i < NT; ++i)
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        double v[2 * R];
                        load(m, i, n, v);
                        addto(G, i, n, w1, v);
                        addto(P2, i, n, w2, v);
                        addto(P3, i, n, w3, v);
                    }
            }
            if constexpr (EXPO == EXPO_COMM) {
                const Mx<S> K = mx_commutator<S>(P2, P3, scr, L);
                mx_each<S>([&](int e) {
                    G.re[e] -= K.im[e];
                    G.im[e] += K.re[e];
                });
                bound = comm_bound(wl, beta);
            } else {
                // -i K of a commutator K is (K_im, -K_re)
                Mx<S> K = mx_commutator<S>(G, P2, scr, L), W, X;
                mx_each<S>([&](int e) {
                    const double r1r = K.im[e], r1i = -K.re[e];
                    W.re[e] = 2.0 * P3.re[e] + r1r;
                    W.im[e] = 2.0 * P3.im[e] + r1i;
                    X.re[e] = (-20.0 * G.re[e] - P3.re[e]) + r1r;
                    X.im[e] = (-20.0 * G.im[e] - P3.im[e]) + r1i;
                });
                K = mx_commutator<S>(G, W, scr, L);
                mx_each<S>([&](int e) {
                    W.re[e] = P2.re[e] - K.im[e] * (1.0 / 60.0);
                    W.im[e] = P2.im[e] + K.re[e] * (1.0 / 60.0);
                });
                K = mx_commutator<S>(X, W, scr, L);
                mx_each<S>([&](int e) {
                    G.re[e] = (G.re[e] + P3.re[e] * (1.0 / 12.0)) + K.im[e] * (1.0 / 240.0);
                    G.im[e] = (G.im[e] + P3.im[e] * (1.0 / 12.0)) - K.re[e] * (1.0 / 240.0);
                });
                bound = m6_bound(wl, beta);
            }
        }
        return G;
    }

    // The bound of this step's exponent(s).
    __device__ __forceinline__ double step_bound() const {
        if constexpr (kRows) {
            auto of = [&](int r) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bounds), 16 * r)); };
            return (double)(S::kPair ? fmaxf(of(tg), of(2 + tg)) : of(tg));
        } else {
            return bound;
        }
    }

    // Scheme q and squarings s of this step; G is scaled by 2^-s.
    __device__ __forceinline__ int plan(Mx<S>& G, int& s) const {
        int q;
        s = 0;
        if constexpr (kRows) {
            const unsigned a = (unsigned)(fits >> (16 * tg)) & 0xffffu;
            const unsigned c = S::kPair ? (unsigned)(fits >> (32 + 16 * tg)) & 0xffffu : a;
            q = a && c && p.force_s < 0 ? max(__builtin_ctz(a), __builtin_ctz(c)) : -1;
        } else {
            q = p.force_s >= 0 ? -1 : plan_scheme(bound, lsth);
        }
        if (q < 0) {
            // squarings: the exponent's own 1-norm may be the smaller bound
            // (terms that cancel)
            plan_scheme_s(p, fmin(step_bound(), mx_norm1<S>(G)), L.lane, lane_sth_of(p, L.lane), q, s);
            s = wave_uniform(s);
            const double sc = ldexp(1.0, -s);
            mx_each<S>([&](int e) {
                G.re[e] *= sc;
                G.im[e] *= sc;
            });
        }
        return wave_uniform(q);
    }

    // E = exp(i G) - I of step t.
    __device__ __forceinline__ Mx<S> slice(int64_t t) {
        Mx<S> G = exponent(t);
        int s;
        const int q = plan(G, s);
        Mx<S> E = mx_expm1<S>(p, G, q, L);
        if (s > 0) mx_square<S>(E, s, scr, L);
        return E;
    }
};

}  // namespace
}  // namespace pm
