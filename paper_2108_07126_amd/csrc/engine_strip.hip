// Propagation on strip teams (mfma_strip.h): FP64, dimensions 33..64.
//
// A block is one team of four waves running a chain of consecutive slices.
// Per slice: the bound sum |w_m| ||B_m||_2 of the lanes' weights picks the
// series' scheme; E = exp(i G) - I; optionally the slice exp(-i G) = I + E^H
// is stored; Q <- Q + E^H Q.  The next slice's exponent is expanded while the
// chain product runs (its basis loads and FMAs go between the products of two
// tile pairs), with the samples of the slice after loaded one slice ahead.
#include "mfma_strip.h"

namespace pm {
namespace {

// The expand step: G = sum_m w_m B_m on the wave's strip (lane m holds w_m),
// in pieces of one tile of one matrix.
template <int NT, int KS>
struct Expand {
    static constexpr int RT = (KS + 3) / 4;
    static constexpr int64_t STR = (int64_t)NT * NT * 512;
    const double* bas;   // the wave's column of tiles (wave-uniform address)
    unsigned off;        // the lane's bytes
    int M;
    double x[2][8];

    __device__ __forceinline__ void load(double (&v)[8], int m, int k) const {
        const char* u = reinterpret_cast<const char*>(bas + m * STR + k * NT * 512);
        const double* b = reinterpret_cast<const double*>(u + off);
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = b[r * 64];
    }
    static __device__ __forceinline__ void add(Strip<NT>& G, int k, double w, const double (&v)[8]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            G.t[k].re[r] = fma(w, v[r], G.t[k].re[r]);
            G.t[k].im[r] = fma(w, v[4 + r], G.t[k].im[r]);
        }
    }
    // Piece f of the first RT matrices (matrix f / RT, tile f % RT): its
    // loads go out, the previous piece's FMAs are done.  Matrices past the
    // basis re-read the last one with their lanes' weight, zero.
    __device__ __forceinline__ void piece(Strip<NT>& G, double wl, int f) {
        if (f < RT * RT) load(x[f & 1], min(f / RT, M - 1), f % RT);
        if (f > 0) {
            const int m = (f - 1) / RT;
            add(G, (f - 1) % RT, readlane_d(wl, m), x[(f - 1) & 1]);
        }
    }
    // The matrices from m0 on, the next one's loads in flight.
    __device__ __forceinline__ void rest(Strip<NT>& G, double wl, int m0) const {
        if (m0 >= M) return;
        double u[RT][8], v[RT][8];
#pragma unroll
        for (int k = 0; k < RT; ++k) load(u[k], m0, k);
        for (int m = m0; m < M; m += 2) {
#pragma unroll
            for (int k = 0; k < RT; ++k) load(v[k], min(m + 1, M - 1), k);
            __builtin_amdgcn_sched_barrier(0);
            const double w0 = readlane_d(wl, m), w1 = readlane_d(wl, m + 1);
#pragma unroll
            for (int k = 0; k < RT; ++k) add(G, k, w0, u[k]);
#pragma unroll
            for (int k = 0; k < RT; ++k) load(u[k], min(m + 2, M - 1), k);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < RT; ++k) add(G, k, w1, v[k]);
        }
    }
};

constexpr int D = 64;

// One wave per SIMD: three operands of the series, the chain product and the
// accumulators (64 registers a strip) take a wave's 512 registers.
template <int KS, bool CH, bool M6, bool JOIN>
__global__ void __launch_bounds__(4 * D) __attribute__((amdgpu_waves_per_eu(1, 1))) propagate_strip(PropParams p) {
    constexpr int NT = D / 16;
    constexpr int RT = (KS + 3) / 4;
    constexpr size_t SB = strip_slot_bytes<NT>();
    extern __shared__ char ssm[];
    float* red = reinterpret_cast<float*>(ssm + 2 * SB);
    int* tick = reinterpret_cast<int*>(red + NT);
    Slots sl{{ssm, ssm + SB}, 0};

    SLane L;
    L.lane = threadIdx.x & 63;
    L.g = L.lane >> 4;
    L.j = L.lane & 15;
    L.c = wave_uniform((int)(threadIdx.x >> 6));

    const int64_t chain = blockIdx.x;
    const int64_t j0 = min(p.n_slices, chain_first(p, chain));
    const int64_t j1 = min(p.n_slices, chain_first(p, chain + 1));
    const int64_t jlast = p.n_slices > 0 ? p.n_slices - 1 : 0;
    WeightRecipe wr;
    if constexpr (M6) wr = m6_recipe(p, L.lane);
    else wr = weight_recipe(p, L.lane);
    auto gather = [&](int64_t j) {
        if constexpr (M6) return m6_gather(p, wr, min(j, jlast));
        else return gather_samples(p, wr, min(j, jlast));
    };
    auto weight = [&](const SliceSamples& v) {
        if constexpr (M6) return m6_weight(p, wr, v);
        else return combine_weight(p, wr, v);
    };
    const double beta = lane_beta_of(p, M6 ? (L.lane & 15) : L.lane);
    const double lsth = lane_sth_of(p, L.lane);
    const double lcth = lane_ctheta_of(p, L.lane);
    Strip<NT> Q = strip_diagonal<NT>(L, 1.0);
    Expand<NT, KS> ex;
    ex.bas = p.basis + mfma_basis_index(D, 0, 0, L.c, 0, 0, 0);
    ex.off = 8u * L.lane;
    ex.M = p.M;
    double wl = weight(gather(j0));
    SliceSamples smp = gather(j0 + 1);
    Strip<NT> G = strip_diagonal<NT>(L, 0.0);
    if constexpr (!M6) ex.rest(G, wl, 0);
    for (int64_t j = j0; j < j1; ++j) {
        double bound;
        if constexpr (M6) {
            Strip<NT> P2 = strip_diagonal<NT>(L, 0.0), P3 = P2;
            G = P2;
            for (int m = 0; m < p.M; ++m) {
                const double w1 = readlane_d(wl, m), w2 = readlane_d(wl, 16 + m), w3 = readlane_d(wl, 32 + m);
#pragma unroll
                for (int k = 0; k < RT; ++k) {
                    double v[8];
                    ex.load(v, m, k);
                    ex.add(G, k, w1, v);
                    ex.add(P2, k, w2, v);
                    ex.add(P3, k, w3, v);
                }
            }
            // G = P1 + P3/12 - (i/240)[-20 P1 - P3 + R1, P2 + R2], R1 = -i[P1, P2],
            // R2 = (i/60)[P1, 2 P3 + R1] (magnus6_exponent); -i K of a commutator K
            // is (K_im, -K_re)
            Strip<NT> K = strip_commutator<NT, KS>(G, P2, L, sl), W, X;
            strip_each<NT>([&](int k, int r) {
                const double r1r = K.t[k].im[r], r1i = -K.t[k].re[r];
                W.t[k].re[r] = 2.0 * P3.t[k].re[r] + r1r;
                W.t[k].im[r] = 2.0 * P3.t[k].im[r] + r1i;
                X.t[k].re[r] = (-20.0 * G.t[k].re[r] - P3.t[k].re[r]) + r1r;
                X.t[k].im[r] = (-20.0 * G.t[k].im[r] - P3.t[k].im[r]) + r1i;
            });
            K = strip_commutator<NT, KS>(G, W, L, sl);
            strip_each<NT>([&](int k, int r) {
                W.t[k].re[r] = P2.t[k].re[r] - K.t[k].im[r] * (1.0 / 60.0);
                W.t[k].im[r] = P2.t[k].im[r] + K.t[k].re[r] * (1.0 / 60.0);
            });
            K = strip_commutator<NT, KS>(X, W, L, sl);
            strip_each<NT>([&](int k, int r) {
                G.t[k].re[r] = (G.t[k].re[r] + P3.t[k].re[r] * (1.0 / 12.0)) + K.t[k].im[r] * (1.0 / 240.0);
                G.t[k].im[r] = (G.t[k].im[r] + P3.t[k].im[r] * (1.0 / 12.0)) - K.t[k].re[r] * (1.0 / 240.0);
            });
            bound = m6_bound(wl, beta);
        } else {
            bound = spectral_bound(wl, beta);
        }
        Strip<NT> E;
        int s = 0;
        auto scale = [&]() {
            const double sc = ldexp(1.0, -s);
            strip_each<NT>([&](int k, int r) {
                G.t[k].re[r] *= sc;
                G.t[k].im[r] *= sc;
            });
        };
        if constexpr (CH) {
            int m;
            plan_cheb_lanes(p, wave_uniform(strip_norm1<NT>(G, L, red)), L.lane, lcth, m, s);
            m = wave_uniform(m);
            s = wave_uniform(s);
            scale();
            E = strip_cheb<NT, KS>(G, m, p.ctheta[m], p.cheb_j + kChebSplitOffset + m * 2 * kChebHalf, L, sl);
        } else {
            int q = p.force_s >= 0 ? -1 : plan_scheme(bound, lsth);
            if (q < 0) {
                // squarings: the exponent's own 1-norm may be the smaller bound
                // (terms that cancel)
                plan_scheme_s(p, fmin(bound, strip_norm1<NT>(G, L, red)), L.lane, lsth, q, s);
                s = wave_uniform(s);
                scale();
            }
            E = strip_expm1<NT, KS>(p, G, wave_uniform(q), L, sl);
        }
        if (s > 0) strip_square<NT, KS>(E, s, L, sl);
        if (p.slices_out) {
            // exp(-i G) = I + E^H: the lane's column of E is a row of the slice
            const int row = 16 * L.c + L.j;
            if (row < p.du) {
                double* out = reinterpret_cast<double*>(p.slices_out) + (j * p.du * p.du + (int64_t)row * p.du) * 2;
                strip_each<NT>([&](int k, int r) {
                    const int col = strip_row(L, k, r);
                    if (col < p.du) {
                        out[2 * col + 0] = E.t[k].re[r] + (row == col ? 1.0 : 0.0);
                        out[2 * col + 1] = -E.t[k].im[r];
                    }
                });
            }
        }
        const char* se = strip_put<NT>(sl, E, L);
        wl = weight(smp);
        smp = gather(j + 2);
        if constexpr (M6) {
            strip_add<NT>(Q, strip_mul<NT, KS>(se, Q, L));
        } else {
            G = strip_diagonal<NT>(L, 0.0);
            strip_add<NT>(Q, strip_mul<NT, KS>(se, Q, L, [&](int f) { ex.piece(G, wl, f); }));
            // (waves past the row tiles form no product, so no piece was loaded
            // for them: their strip of G stays zero, as the 1-norm takes it)
            if (L.c < RT) ex.piece(G, wl, RT * RT);
            ex.rest(G, wl, RT);
        }
    }
    if (p.chain_out && chain < p.n_chains) strip_node_store<NT>(p.chain_out + chain * (int64_t)D * D * 2, Q, L);
    strip_tree<NT, KS, JOIN>(p, blockIdx.x, Q, L, sl, tick);
}

template <int KS, bool CH, bool M6, bool JOIN>
hipError_t launch_strip_one(const PropParams& p, hipStream_t stream) {
    constexpr size_t lds = 2 * strip_slot_bytes<D / 16>() + 64;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)propagate_strip<KS, CH, M6, JOIN>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((propagate_strip<KS, CH, M6, JOIN>), dim3((unsigned)p.n_leaves), dim3(4 * D), lds, stream, p);
    return hipGetLastError();
}

// The Taylor series of orders 2, 4 and CF4 over the k-slices the dimension
// reaches, in steps of two.  Chains of fewer than four slices leave most products to
// the tree, which joins their nodes (64 levels, 100 slices: error 1.2e-15 in 132 us,
// without 1.5e-14 in 129 us); longer chains hold the rounding down themselves
// (1000 slices 259 us, joined 264 us).
template <int KS>
hipError_t launch_strip_ks(const PropParams& p, hipStream_t stream) {
    if constexpr (KS < D / 4) {
        if (p.du > 4 * KS) return launch_strip_ks<KS + 2>(p, stream);
    }
    return p.chunk < 4 ? launch_strip_one<KS, false, false, true>(p, stream)
                       : launch_strip_one<KS, false, false, false>(p, stream);
}

}  // namespace

// (The Chebyshev series runs over three quarters or all of the k-slices, the
// sixth-order scheme over all; the series' truncation is larger than the tree's
// rounding.)
hipError_t launch_strip(const PropParams& p, hipStream_t stream) {
    const bool ch = p.method == PM_EXPM_CHEBYSHEV;
    if (p.order == kOrderM6)
        return ch ? launch_strip_one<16, true, true, false>(p, stream)
                  : launch_strip_one<16, false, true, true>(p, stream);
    if (ch)
        return p.du <= 48 ? launch_strip_one<12, true, false, false>(p, stream)
                          : launch_strip_one<16, true, false, false>(p, stream);
    return launch_strip_ks<10>(p, stream);
}

}  // namespace pm
