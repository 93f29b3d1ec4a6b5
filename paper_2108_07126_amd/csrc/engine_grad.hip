// Adjoint gradient of a real loss L(U(T)) with respect to every control
// sample, on the MFMA tile engine in FP64.
//
// With W the loss gradient in the convention dL = Re Tr(W^H dU(T)),
// P_j = U_{j-1} ... U_0 and S_j = U_{N-1} ... U_{j+1}:
//     dL = Re sum_j Tr(W^H S_j dU_j P_j) = Re sum_j Tr(F_j dG_j),
//     F_j = L_f(G_j, Lambda_j),  Lambda_j = P_j W^H S_j,  f(G) = exp(-i G),
// (cyclic trace and Tr(A L_f(G, E)) = Tr(L_f(G, A) E)), so that
//     dL / dw_{j,m} = Re Tr(F_j B_m)
// for the expand step's weights; the chain rule through the weight formulas
// gives dL / d samples.  The prefix/suffix structure is carried by
//     Omega_j = P_j W^H (U_{N-1} ... U_j),  Lambda_j = Omega_j U_j^H,
//     Omega_{j+1} = U_j Omega_j U_j^H,
// started at each chain from its checkpoint P_{j0}: the forward pass (run
// just before, with every tree node kept) leaves the product of every aligned
// power-of-two range of blocks, and P_{j0} is assembled from at most
// log2(#blocks) of them plus the earlier chains of its own block; then
// Omega_{j0} = P Z P^H with Z = W^H U(T) (P unitary).  Inside a chain the
// slices are recomputed (a checkpoint every `chunk` slices, nothing else
// stored).  F_j is the upper-right block of exp(-i [[G, Lambda], [0, G]]),
// evaluated with the same cos/sin Taylor scheme and scaling-and-squaring as
// the forward pass on (value, derivative) pairs:
//     (A, dA)(B, dB) = (A B, A dB + dA B).
#include "mfma_tiles.h"

namespace pm {
namespace {

template <class G>
__device__ __forceinline__ Tile<double> load_user(const double* A, int du, double pad_diag,
                                                  const Lane& L) {
    Tile<double> t;
    const int col = 16 * L.TJ + L.j;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * L.TI + crow<double>(L.g, r);
        if (row < du && col < du) {
            t.re[r] = A[(row * du + col) * 2 + 0];
            t.im[r] = A[(row * du + col) * 2 + 1];
        } else {
            t.re[r] = (row == col) ? pad_diag : 0.0;
            t.im[r] = 0.0;
        }
    }
    return t;
}

// The conjugate transpose of a tile set, stored into a slot.
template <class G>
__device__ __forceinline__ void slot_store_adj(double* slot, const Tile<double>& t, const Lane& L) {
    double* re = slot;
    double* im = slot + G::PLANE;
    const int col = 16 * L.TJ + L.j;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * L.TI + crow<double>(L.g, r);
        re[col * G::LD + row] = t.re[r];
        im[col * G::LD + row] = -t.im[r];
    }
}

__device__ __forceinline__ Tile<double> tadd(const Tile<double>& a, const Tile<double>& b) {
    Tile<double> c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        c.re[r] = a.re[r] + b.re[r];
        c.im[r] = a.im[r] + b.im[r];
    }
    return c;
}

__device__ __forceinline__ Tile<double> tzero() {
    Tile<double> c;
#pragma unroll
    for (int r = 0; r < 4; ++r) c.re[r] = c.im[r] = 0.0;
    return c;
}

__device__ __forceinline__ Tile<double> tscale(const Tile<double>& a, int e) {
    Tile<double> c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        c.re[r] = ldexp(a.re[r], e);
        c.im[r] = ldexp(a.im[r], e);
    }
    return c;
}

// C - i S
__device__ __forceinline__ Tile<double> c_minus_is(const Tile<double>& C, const Tile<double>& S) {
    Tile<double> u;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        u.re[r] = C.re[r] + S.im[r];
        u.im[r] = C.im[r] - S.re[r];
    }
    return u;
}

template <class G>
__device__ __forceinline__ Tile<double> mul2(const Tile<double>& A, const Tile<double>& B,
                                             const Lane& L, double* s0, double* s1) {
    team_sync<G>();
    slot_store<G, double>(s0, A, L);
    slot_store<G, double>(s1, B, L);
    team_sync<G>();
    return slot_mul<G, double>(s0, s1, L);
}

// A B^H
template <class G>
__device__ __forceinline__ Tile<double> mul_adjB(const Tile<double>& A, const Tile<double>& B,
                                                 const Lane& L, double* s0, double* s1) {
    team_sync<G>();
    slot_store<G, double>(s0, A, L);
    slot_store_adj<G>(s1, B, L);
    team_sync<G>();
    return slot_mul<G, double>(s0, s1, L);
}

// A^H B
template <class G>
__device__ __forceinline__ Tile<double> mul_adjA(const Tile<double>& A, const Tile<double>& B,
                                                 const Lane& L, double* s0, double* s1) {
    team_sync<G>();
    slot_store_adj<G>(s0, A, L);
    slot_store<G, double>(s1, B, L);
    team_sync<G>();
    return slot_mul<G, double>(s0, s1, L);
}

// (exp(-i G), L_f(G, E)) by the degree-m cos/sin Taylor scheme on
// (value, derivative) pairs; G and E pre-scaled by 2^-s.
template <class G>
__device__ void pair_taylor(const Tile<double>& Gt, const Tile<double>& Et, int m, const Lane& L,
                            double* s0, double* s1, Tile<double>& U, Tile<double>& dU) {
    Tile<double> C = ident<double>(L), dC = tzero(), S, dS;
    if (m <= 1) {
        S = Gt;
        dS = Et;
    } else {
        const int qc = m / 2, qs = (m - 1) / 2;
        team_sync<G>();
        slot_store<G, double>(s0, Gt, L);
        slot_store<G, double>(s1, Et, L);
        team_sync<G>();
        const Tile<double> Y = slot_mul<G, double>(s0, s0, L);
        const Tile<double> dY = tadd(slot_mul<G, double>(s0, s1, L), slot_mul<G, double>(s1, s0, L));
        Tile<double> Sp = ident<double>(L), dSp = tzero();
        axpy(C, cos_coef(1), Y);
        axpy(dC, cos_coef(1), dY);
        if (qs >= 1) {
            axpy(Sp, sin_coef(1), Y);
            axpy(dSp, sin_coef(1), dY);
        }
        Tile<double> P = Y, dP = dY;
        for (int k = 2; k <= qc; ++k) {
            team_sync<G>();
            slot_store<G, double>(s0, P, L);
            slot_store<G, double>(s1, Y, L);
            team_sync<G>();
            const Tile<double> Pn = slot_mul<G, double>(s0, s1, L);
            team_sync<G>();
            slot_store<G, double>(s1, dY, L);
            team_sync<G>();
            const Tile<double> t1 = slot_mul<G, double>(s0, s1, L);   // P dY
            team_sync<G>();
            slot_store<G, double>(s0, dP, L);
            slot_store<G, double>(s1, Y, L);
            team_sync<G>();
            const Tile<double> t2 = slot_mul<G, double>(s0, s1, L);   // dP Y
            P = Pn;
            dP = tadd(t1, t2);
            axpy(C, cos_coef(k), P);
            axpy(dC, cos_coef(k), dP);
            if (k <= qs) {
                axpy(Sp, sin_coef(k), P);
                axpy(dSp, sin_coef(k), dP);
            }
        }
        if (qs >= 1) {
            team_sync<G>();
            slot_store<G, double>(s0, Gt, L);
            slot_store<G, double>(s1, Sp, L);
            team_sync<G>();
            S = slot_mul<G, double>(s0, s1, L);
            team_sync<G>();
            slot_store<G, double>(s1, dSp, L);
            team_sync<G>();
            const Tile<double> t1 = slot_mul<G, double>(s0, s1, L);   // G dS'
            team_sync<G>();
            slot_store<G, double>(s0, Et, L);
            slot_store<G, double>(s1, Sp, L);
            team_sync<G>();
            const Tile<double> t2 = slot_mul<G, double>(s0, s1, L);   // E S'
            dS = tadd(t1, t2);
        } else {
            S = Gt;
            dS = Et;
        }
    }
    U = c_minus_is(C, S);
    dU = c_minus_is(dC, dS);
}

// U_j = exp(-i G) from the scaled exponent Gt by the series and s squarings.
template <class G>
__device__ __forceinline__ Tile<double> slice_exp(const Tile<double>& Gt, int m, int s, const Lane& L, double* s0,
                                                  double* s1) {
    return square_n<G, double>(taylor_exp<G, double>(Gt, m, L, s0, s1), s, L, s0);
}

// Sum over the team of a per-lane value; uniform result.  red: LDS, TW doubles.
template <class G>
__device__ __forceinline__ double team_sum(double x, const Lane& L, double* red) {
    x = row16_sum(x);
    x = readlane_d(x, 0) + readlane_d(x, 16) + readlane_d(x, 32) + readlane_d(x, 48);
    if constexpr (G::TW == 1) {
        return x;
    } else {
        __syncthreads();
        if (L.lane == 0) red[L.wt] = x;
        __syncthreads();
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < G::TW; ++w) t += red[w];
        return t;
    }
}

// The product of every slice before `chain` (U_{j0-1} ... U_0) from a forward
// pass that kept its tree nodes and chain products: the aligned
// power-of-two node ranges over the blocks before this one (earliest range
// first), then this block's earlier chains.
template <class G>
__device__ Tile<double> chain_checkpoint(const PropParams& p, int64_t chain, const Lane& L, double* s0,
                                         double* s1) {
    const int64_t NN = (int64_t)G::D * G::D * 2;
    Tile<double> P = ident<double>(L);
    // leaves [0, b) as aligned tree nodes, earliest first: at level l the
    // first d_l nodes of b's group, d_l the base-kFanIn digit l of b
    const int64_t b = chain / p.chains_per_leaf;
    int nlev = 0;
    for (int64_t cnt = p.n_leaves; cnt > 1; cnt = (cnt + kFanIn - 1) / kFanIn) ++nlev;
    for (int l = nlev; l >= 0; --l) {
        const int64_t d = (b >> (kFanInLog2 * l)) & (kFanIn - 1);
        if (d == 0) continue;
        int64_t off = 0, cnt = p.n_leaves;
        for (int q = 0; q < l; ++q) {
            off += cnt;
            cnt = (cnt + kFanIn - 1) / kFanIn;
        }
        const int64_t first = (b >> (kFanInLog2 * (l + 1))) << kFanInLog2;
        for (int64_t k = 0; k < d; ++k)
            P = mul2<G>(node_load<G>(p.nodes + (off + first + k) * NN, L), P, L, s0, s1);
    }
    for (int64_t c = b * p.chains_per_leaf; c < chain; ++c)
        P = mul2<G>(node_load<G>(p.chain_out + c * NN, L), P, L, s0, s1);
    return P;
}

template <int D, int NT, bool BL>
__global__ void __launch_bounds__(64 * (D / 16) * (D / 16) * NT)
__attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2, 8)))
backward_mfma(GradParams gp) {
    using G = Geo<D, NT>;
    const PropParams& p = gp.p;
    extern __shared__ double dsm[];
    double* slots = dsm;
    double* red = slots + NT * 2 * G::SLOT;
    double* lbasis = red + G::TD * D + 2;

    Lane L;
    L.lane = threadIdx.x & 63;
    L.g = L.lane >> 4;
    L.j = L.lane & 15;
    const int wave = wave_uniform((int)(threadIdx.x >> 6));
    const int team = wave / G::TW;
    L.wt = wave % G::TW;
    L.TI = L.wt / G::TD;
    L.TJ = L.wt % G::TD;
    L.ks = (p.du + 3) / 4;   // the tiles vanish outside the leading du x du block
    double* s0 = slots + team * 2 * G::SLOT;
    double* s1 = s0 + G::SLOT;
    if constexpr (BL) {
        const int n = p.M * G::TW * 512;
        block_copy_to_lds(lbasis, p.basis, n);
        __syncthreads();
    }
    const double* bas = BL ? lbasis : p.basis;
    // backward unit: part `part` of chain `chain` (split parts of equal length)
    const int64_t unit = (int64_t)blockIdx.x * NT + team;
    const int64_t chain = unit / gp.split;
    const int64_t part = unit % gp.split;
    if (chain >= p.n_chains) return;   // no block-wide barrier follows
    const int64_t c0 = chain * p.chunk, c1 = min(p.n_slices, c0 + p.chunk);
    const int64_t sub = (p.chunk + gp.split - 1) / gp.split;
    const int64_t j0 = min(c1, c0 + part * sub);
    const int64_t j1 = min(c1, j0 + sub);
    if (j0 >= j1) return;

    const WeightRecipe wr = weight_recipe(p, L.lane);
    const double lth = lane_theta_of(p, L.lane);
    const int64_t bofs = mfma_basis_index(D, 0, L.TI, L.TJ, 0, 0, L.lane);
    // slice j's exponent, scaled by 2^-s for its plan (m, s)
    auto slice_exponent = [&](const SliceSamples& smp, Tile<double>& Gt, int& m, int& s) {
        const double wl = combine_weight(p, wr, smp);
        double gre[4] = {0, 0, 0, 0}, gim[4] = {0, 0, 0, 0};
#pragma unroll 4
        for (int mm = 0; mm < p.M; ++mm) {
            const double w = readlane_d(wl, mm);
            const double* bb = bas + bofs + (int64_t)mm * G::TW * 512;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                gre[r] = fma(w, bb[r * 64], gre[r]);
                gim[r] = fma(w, bb[256 + r * 64], gim[r]);
            }
        }
        const double nu = wave_uniform(team_norm1<G, double>(gre, gim, L, red));
        plan_expm_lanes(p, nu, L.lane, lth, m, s);
        m = wave_uniform(m);
        s = wave_uniform(s);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            Gt.re[r] = ldexp(gre[r], -s);
            Gt.im[r] = ldexp(gim[r], -s);
        }
    };

    // checkpoint P = U_{j0-1} ... U_0: the chain's, then the unit's
    // predecessors in the chain recomputed
    Tile<double> P = chain_checkpoint<G>(p, chain, L, s0, s1);
    for (int64_t j = c0; j < j0; ++j) {
        Tile<double> Gt;
        int m, s;
        slice_exponent(gather_samples(p, wr, j), Gt, m, s);
        const Tile<double> U = slice_exp<G>(Gt, m, s, L, s0, s1);
        P = mul2<G>(U, P, L, s0, s1);
    }
    // Omega_{j0} = P Z P^H, Z = W^H U(T)
    const Tile<double> Wt = load_user<G>(gp.W, p.du, 0.0, L);
    const Tile<double> UTt = load_user<G>(gp.UT, p.du, 1.0, L);
    const Tile<double> Z = mul_adjA<G>(Wt, UTt, L, s0, s1);
    Tile<double> Om = mul_adjB<G>(mul2<G>(P, Z, L, s0, s1), P, L, s0, s1);

    SliceSamples smp = gather_samples(p, wr, j0);
    for (int64_t j = j0; j < j1; ++j) {
        const SliceSamples cur = smp;
        if (j + 1 < j1) smp = gather_samples(p, wr, j + 1);
        Tile<double> Gt;
        int m, s;
        slice_exponent(cur, Gt, m, s);
        // U_j, Lambda_j = Omega_j U_j^H and Omega_{j+1} = U_j Omega_j U_j^H =
        // U_j Lambda_j
        const Tile<double> U = slice_exp<G>(Gt, m, s, L, s0, s1);
        const Tile<double> Lam = mul_adjB<G>(Om, U, L, s0, s1);
        Om = mul2<G>(U, Lam, L, s0, s1);
        // F_j = L_f(G_j, Lambda_j)
        Tile<double> Up, F;
        pair_taylor<G>(Gt, tscale(Lam, -s), m, L, s0, s1, Up, F);
        for (int q = 0; q < s; ++q) {
            team_sync<G>();
            slot_store<G, double>(s0, Up, L);
            slot_store<G, double>(s1, F, L);
            team_sync<G>();
            const Tile<double> Un = slot_mul<G, double>(s0, s0, L);
            F = tadd(slot_mul<G, double>(s0, s1, L), slot_mul<G, double>(s1, s0, L));
            Up = Un;
        }
        // dL/dw_{j,m} = Re Tr(F B_m) = sum over entries of Re(F) Re(B) + Im(F) Im(B) (B Hermitian)
        for (int mm = 0; mm < p.M; ++mm) {
            const double* bb = bas + bofs + (int64_t)mm * G::TW * 512;
            double part = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) part = fma(F.re[r], bb[r * 64], fma(F.im[r], bb[256 + r * 64], part));
            const double g = team_sum<G>(part, L, red);
            if (L.lane == 0 && L.wt == 0) gp.gw[j * p.M + mm] = g;
        }
    }
}

// Rows < rows and columns < cols of a tile set from a row-major complex
// block with leading dimension ld (zero elsewhere).
template <class G>
__device__ __forceinline__ Tile<double> load_block(const double* A, int rows, int cols, int ld, const Lane& L) {
    Tile<double> t;
    const int col = 16 * L.TJ + L.j;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * L.TI + crow<double>(L.g, r);
        const bool in = row < rows && col < cols;
        t.re[r] = in ? A[(row * ld + col) * 2 + 0] : 0.0;
        t.im[r] = in ? A[(row * ld + col) * 2 + 1] : 0.0;
    }
    return t;
}

template <class G>
__device__ __forceinline__ void store_block(double* A, const Tile<double>& t, int rows, int cols, int ld,
                                            const Lane& L) {
    const int col = 16 * L.TJ + L.j;
    if (col >= cols) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * L.TI + crow<double>(L.g, r);
        if (row < rows) {
            A[(row * ld + col) * 2 + 0] = t.re[r];
            A[(row * ld + col) * 2 + 1] = t.im[r];
        }
    }
}

// Trajectory: every prefix P_j = U_{j-1} ... U_0, j = 0..N (applied to a
// block of states, or to a density matrix), from the same checkpoints as the
// gradient: each chain starts from its checkpoint and multiplies its
// recomputed slices in, writing its rows of the output before each slice;
// the last chain also writes j = N.
template <int D, int NT, bool BL>
__global__ void __launch_bounds__(64 * (D / 16) * (D / 16) * NT)
__attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2, 8)))
trajectory_mfma(TrajParams tp) {
    using G = Geo<D, NT>;
    const PropParams& p = tp.p;
    extern __shared__ double dsm[];
    double* slots = dsm;
    double* red = slots + NT * 2 * G::SLOT;
    double* lbasis = red + G::TD * D + 2;

    Lane L;
    L.lane = threadIdx.x & 63;
    L.g = L.lane >> 4;
    L.j = L.lane & 15;
    const int wave = wave_uniform((int)(threadIdx.x >> 6));
    const int team = wave / G::TW;
    L.wt = wave % G::TW;
    L.TI = L.wt / G::TD;
    L.TJ = L.wt % G::TD;
    L.ks = (tp.p.du + 3) / 4;   // the tiles vanish outside the leading du x du block
    double* s0 = slots + team * 2 * G::SLOT;
    double* s1 = s0 + G::SLOT;
    if constexpr (BL) {
        const int n = p.M * G::TW * 512;
        block_copy_to_lds(lbasis, p.basis, n);
        __syncthreads();
    }
    const double* bas = BL ? lbasis : p.basis;
    const int64_t chain = (int64_t)blockIdx.x * NT + team;
    if (chain >= p.n_chains) return;   // no block-wide barrier follows
    const int64_t j0 = chain * p.chunk;
    const int64_t j1 = min(p.n_slices, j0 + p.chunk);
    const int du = p.du;
    const int cols = tp.kind == PM_TRAJ_STATES ? tp.n_vec : du;
    const int64_t stride = (int64_t)du * cols * 2;

    // S_j: P_j, P_j Psi_0 or P_j rho_0 P_j^H at the chain's first slice
    Tile<double> S = chain_checkpoint<G>(p, chain, L, s0, s1);
    if (tp.kind == PM_TRAJ_STATES) {
        S = mul2<G>(S, load_block<G>(tp.x0, du, cols, cols, L), L, s0, s1);
    } else if (tp.kind == PM_TRAJ_DENSITY) {
        S = mul_adjB<G>(mul2<G>(S, load_block<G>(tp.x0, du, du, du, L), L, s0, s1), S, L, s0, s1);
    }
    const WeightRecipe wr = weight_recipe(p, L.lane);
    const double lth = lane_theta_of(p, L.lane);
    SliceSamples smp = gather_samples(p, wr, j0);
    const int64_t bofs = mfma_basis_index(D, 0, L.TI, L.TJ, 0, 0, L.lane);
    // the commutator-free scheme has two exponentials per slice: a slice
    // boundary is every second one
    const int vs = p.order == kOrderCF4 ? 1 : 0;
    for (int64_t j = j0; j < j1; ++j) {
        if ((j & vs) == 0) store_block<G>(tp.out + (j >> vs) * stride, S, du, cols, cols, L);
        const double wl = combine_weight(p, wr, smp);
        if (j + 1 < j1) smp = gather_samples(p, wr, j + 1);
        double gre[4] = {0, 0, 0, 0}, gim[4] = {0, 0, 0, 0};
#pragma unroll 4
        for (int m = 0; m < p.M; ++m) {
            const double w = readlane_d(wl, m);
            const double* bb = bas + bofs + (int64_t)m * G::TW * 512;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                gre[r] = fma(w, bb[r * 64], gre[r]);
                gim[r] = fma(w, bb[256 + r * 64], gim[r]);
            }
        }
        const double nu = wave_uniform(team_norm1<G, double>(gre, gim, L, red));
        int m, s;
        plan_expm_lanes(p, nu, L.lane, lth, m, s);
        m = wave_uniform(m);
        s = wave_uniform(s);
        Tile<double> Gt;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            Gt.re[r] = ldexp(gre[r], -s);
            Gt.im[r] = ldexp(gim[r], -s);
        }
        const Tile<double> U = slice_exp<G>(Gt, m, s, L, s0, s1);
        S = mul2<G>(U, S, L, s0, s1);
        if (tp.kind == PM_TRAJ_DENSITY) S = mul_adjB<G>(S, U, L, s0, s1);
    }
    if (j1 == p.n_slices) store_block<G>(tp.out + (p.n_slices >> vs) * stride, S, du, cols, cols, L);
}

// dL/d samples from dL/dw by the weight formulas of the expand step; one
// thread per (control, sample).
__global__ void __launch_bounds__(256) samples_grad(GradParams gp, double* grad) {
    const PropParams& p = gp.p;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int K = p.K, M = p.M;
    const int64_t S = p.n_samples, N = p.n_slices;
    if (idx >= (int64_t)K * S) return;
    const int k = (int)(idx / S);
    const int64_t q = idx % S;
    const double h = p.h, h2 = h * h * (1.0 / 12.0);
    const double* g = gp.gw;
    const double* c = p.samples;
    if (p.order == 2) {
        grad[idx] = h * g[q * M + 1 + k];
        return;
    }
    if (p.order == kOrderCF4) {
        // exponents 2j and 2j+1 weigh the samples of slice j by
        // (h/12)(3, 4, -1) and (h/12)(-1, 4, 3)
        const double h12 = h * (1.0 / 12.0);
        const int64_t NS = N >> 1;
        double a = 0.0;
        if (q & 1) {
            const int64_t j = (q - 1) / 2;
            a = 4.0 * (g[(2 * j) * M + 1 + k] + g[(2 * j + 1) * M + 1 + k]);
        } else {
            const int64_t jf = q / 2, jl = q / 2 - 1;   // first sample of jf, last of jl
            if (jf < NS) a += 3.0 * g[(2 * jf) * M + 1 + k] - g[(2 * jf + 1) * M + 1 + k];
            if (jl >= 0) a += 3.0 * g[(2 * jl + 1) * M + 1 + k] - g[(2 * jl) * M + 1 + k];
        }
        grad[idx] = h12 * a;
        return;
    }
    double acc = 0.0;
    // role 1 (middle sample of slice (q-1)/2)
    if (q & 1) {
        const int64_t j = (q - 1) / 2;
        acc += (4.0 * h / 6.0) * g[j * M + 1 + k];
    } else {
        // role 0 of slice q/2 and role 2 of slice q/2 - 1
        for (int role = 0; role < 2; ++role) {
            const int64_t j = role == 0 ? q / 2 : q / 2 - 1;
            if (j < 0 || j >= N) continue;
            const double* gj = g + j * M;
            const double sg = role == 0 ? -1.0 : 1.0;   // d(s2 - s0)
            acc += (h / 6.0) * gj[1 + k] + sg * h2 * gj[1 + K + k];
            int mq = 1 + 2 * K;
            for (int a = 0; a < K; ++a)
                for (int b = a + 1; b < K; ++b, ++mq) {
                    // w = h2 (s0_a s2_b - s2_a s0_b)
                    const double* ca = c + (int64_t)a * S + 2 * j;
                    const double* cb = c + (int64_t)b * S + 2 * j;
                    if (a == k) acc += gj[mq] * h2 * (role == 0 ? cb[2] : -cb[0]);
                    if (b == k) acc += gj[mq] * h2 * (role == 0 ? -ca[2] : ca[0]);
                }
        }
    }
    grad[idx] = acc;
}

template <int D, int NT, bool BL>
hipError_t launch_bwd(const GradParams& gp, size_t lds, hipStream_t stream) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)backward_mfma<D, NT, BL>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int64_t blocks = (gp.p.n_chains * gp.split + NT - 1) / NT;
    hipLaunchKernelGGL((backward_mfma<D, NT, BL>), dim3((unsigned)blocks), dim3(64 * (D / 16) * (D / 16) * NT),
                       lds, stream, gp);
    return hipGetLastError();
}

template <int D, int NT, bool BL>
hipError_t launch_traj(const TrajParams& tp, size_t lds, hipStream_t stream) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)trajectory_mfma<D, NT, BL>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int64_t blocks = (tp.p.n_chains + NT - 1) / NT;
    hipLaunchKernelGGL((trajectory_mfma<D, NT, BL>), dim3((unsigned)blocks), dim3(64 * (D / 16) * (D / 16) * NT),
                       lds, stream, tp);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_adjoint_wave16(const GradParams& gp, hipStream_t stream);
hipError_t launch_adjoint_wave32(const GradParams& gp, hipStream_t stream);
hipError_t launch_trajectory_wave16(const TrajParams& tp, hipStream_t stream);
hipError_t launch_trajectory_wave32(const TrajParams& tp, hipStream_t stream);

// LDS of the 64-wide kernels: two staging slots and the reduction rows.
constexpr size_t kWide64Lds = sizeof(double) * (2 * Geo<64, 1>::SLOT + 4 * 64 + 2);

hipError_t launch_trajectory(int D, const TrajParams& tp, hipStream_t stream) {
    switch (D) {
        case 16: return launch_trajectory_wave16(tp, stream);
        case 32: return launch_trajectory_wave32(tp, stream);
        case 64: return launch_traj<64, 1, false>(tp, kWide64Lds, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_backward(int D, const GradParams& gp, double* grad_samples, hipStream_t stream) {
    hipError_t e;
    // one-wave teams write dL/d samples themselves at order 2
    GradParams gq = gp;
    gq.grad_direct = (D <= 32 && gp.p.order == 2) ? grad_samples : nullptr;
    switch (D) {
        case 16: e = launch_adjoint_wave16(gq, stream); break;
        case 32: e = launch_adjoint_wave32(gq, stream); break;
        case 64: e = launch_bwd<64, 1, false>(gp, kWide64Lds, stream); break;
        default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)gp.p.K * gp.p.n_samples;
    if (n == 0 || gq.grad_direct) return hipSuccess;
    hipLaunchKernelGGL(samples_grad, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, gq,
                       grad_samples);
    return hipGetLastError();
}

}  // namespace pm
