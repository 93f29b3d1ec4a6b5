// One-wave teams: the FP64 MFMA engine of dimensions 5..32.
//
// One wave carries a chain and holds every D x D complex matrix, D = 16 NT, in
// registers: NT x NT tiles of 16 x 16 in the accumulator layout of
// v_mfma_f64_16x16x4f64 (lane 16 g + j holds rows g + 4 r, r = 0..3, of column
// j of each tile).  Register r of tile (k, n) is the B operand of a k-slice as it
// stands, and register r of tile (k, i) of S the A operand of S^H: a product
// S^H X takes both operands from the lane's own registers.  So the engine
// computes S^H X only: S X for the Hermitian factors of the series, and for
// the chain it carries E = exp(i G) - I, whose adjoint is exp(-i G) - I:
// Q <- Q + E^H Q.  No product touches LDS and no wave waits for another one.
//
// KS: the k-slices (of four rows) that the embedded dimension reaches,
// du <= 4 KS; rows and columns past them are zero in every product.
#pragma once

#include "mfma_tiles.h"

namespace pm {
namespace {

template <int NT>
struct Sq {
    Tile<double> t[NT][NT];   // [row tile][column tile]
};

struct WLane {
    int lane, g, j;
};

// f(row tile, column tile, register) over the entries a lane holds.
template <int NT, class F>
__device__ __forceinline__ void sq_each(F f) {
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) f(i, n, r);
}

__device__ __forceinline__ bool sq_diag(const WLane& L, int i, int n, int r) { return i == n && L.g + 4 * r == L.j; }

template <int NT>
__device__ __forceinline__ Sq<NT> sq_diagonal(const WLane& L, double v) {
    Sq<NT> s;
    sq_each<NT>([&](int i, int n, int r) {
        s.t[i][n].re[r] = sq_diag(L, i, n, r) ? v : 0.0;
        s.t[i][n].im[r] = 0.0;
    });
    return s;
}

template <int NT>
__device__ __forceinline__ void sq_add(Sq<NT>& y, const Sq<NT>& x) {
    sq_each<NT>([&](int i, int n, int r) {
        y.t[i][n].re[r] += x.t[i][n].re[r];
        y.t[i][n].im[r] += x.t[i][n].im[r];
    });
}

// S^H X as three real products chained through the accumulator:
// k = (Sr - Si) Xr, Re = k + Si (Xr + Xi), Im = k + Sr (Xi - Xr).  Re and Im
// start from k as their MFMAs' C operand, so no sums follow the matrix
// instructions (the usual t1 + t2, t3 - t1 + t2 take 12 more vector
// instructions a tile, and none of those overlaps an FP64 MFMA of its SIMD).
// STK (NT = 1): slice pairs.  The two 8 x 8 diagonal blocks hold two slices
// and are multiplied as the stacked product [A_a; A_b] [B_a, B_b], K = 8
// instead of 16: for k-slice s the lane (g, j) supplies its register s (its
// column in the first block) or s + 2 (second block) of both operands.  The
// off-diagonal blocks of the result hold cross products, which no stacked
// product reads (pair_mask clears them before a full one).
template <int NT, int KS, bool STK = false>
__device__ __forceinline__ Sq<NT> sq_mul(const Sq<NT>& S, const Sq<NT>& X) {
    Sq<NT> out;
    if constexpr (STK) {
        static_assert(NT == 1, "slice pairs live in one tile");
        const bool hi = (__lane_id() & 8) != 0;
        const Tile<double>&A = S.t[0][0], &B = X.t[0][0];
        double sr[2], si[2], xr[2], xi[2];
        d4_t kk = {0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            sr[q] = hi ? A.re[q + 2] : A.re[q];
            si[q] = hi ? A.im[q + 2] : A.im[q];
            xr[q] = hi ? B.re[q + 2] : B.re[q];
            xi[q] = hi ? B.im[q + 2] : B.im[q];
            kk = mfma16(sr[q] - si[q], xr[q], kk);
        }
        d4_t re = kk, im = kk;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            re = mfma16(si[q], xr[q] + xi[q], re);
            im = mfma16(sr[q], xi[q] - xr[q], im);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            out.t[0][0].re[r] = re[r];
            out.t[0][0].im[r] = im[r];
        }
        return out;
    } else {
        constexpr int RT = (KS + 3) / 4;
        // the operands' sums ahead of the MFMAs (one right before the MFMA
        // that reads it would cost wait states each time)
        double sd[NT][KS];
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int q = 0; q < KS; ++q) sd[i][q] = S.t[q >> 2][i].re[q & 3] - S.t[q >> 2][i].im[q & 3];
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            double xp[KS], xm[KS];
#pragma unroll
            for (int q = 0; q < KS; ++q) {
                const Tile<double>& B = X.t[q >> 2][n];
                xp[q] = B.re[q & 3] + B.im[q & 3];
                xm[q] = B.im[q & 3] - B.re[q & 3];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                d4_t kk = {0, 0, 0, 0};
                if (i < RT && n < RT) {
#pragma unroll
                    for (int q = 0; q < KS; ++q) kk = mfma16(sd[i][q], X.t[q >> 2][n].re[q & 3], kk);
                }
                d4_t re = kk, im = kk;
                if (i < RT && n < RT) {
#pragma unroll
                    for (int q = 0; q < KS; ++q) {
                        const Tile<double>& A = S.t[q >> 2][i];
                        re = mfma16(A.im[q & 3], xp[q], re);
                        im = mfma16(A.re[q & 3], xm[q], im);
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    out.t[i][n].re[r] = re[r];
                    out.t[i][n].im[r] = im[r];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        return out;
    }
}

// exp(i G) - I for the (pre-scaled) Hermitian G by evaluation scheme q
// (scheme_degree(q); coefficients p.tc[k] = 1/k!, zero past the degree cap),
// Paterson-Stockmeyer in blocks of three powers with Y = G G, Z = G Y:
//   q = 0  i G;   q = 1  i G - Y/2;   q = 2  i G - Y (1/2 + i G/6 - Y/24);
//   q >= 3 blocks B_i = c_{3i} + c_{3i+1} i G - c_{3i+2} Y over powers of
//          (i G)^3 = -i Z, X <- B_i - i Z X: q products in all.
// Every left factor is Hermitian.
template <int NT, int KS, bool STK>
__device__ __forceinline__ Sq<NT> sq_expm1(const PropParams& p, const Sq<NT>& G, int q, const WLane& L) {
    Sq<NT> E;
    if (q == 0) {
        sq_each<NT>([&](int i, int n, int r) {
            E.t[i][n].re[r] = -G.t[i][n].im[r];
            E.t[i][n].im[r] = G.t[i][n].re[r];
        });
        return E;
    }
    const Sq<NT> Y = sq_mul<NT, KS, STK>(G, G);
    // c0 I + c1 i G - c2 Y into E
    auto block = [&](double c0, double c1, double c2) {
        sq_each<NT>([&](int i, int n, int r) {
            E.t[i][n].re[r] = fma(-c1, G.t[i][n].im[r], fma(-c2, Y.t[i][n].re[r], sq_diag(L, i, n, r) ? c0 : 0.0));
            E.t[i][n].im[r] = fma(c1, G.t[i][n].re[r], -c2 * Y.t[i][n].im[r]);
        });
    };
    if (q <= 2) {
        if (q == 1) {
            block(0.0, 1.0, p.tc[2]);
            return E;
        }
        block(p.tc[2], p.tc[3], p.tc[4]);
        E = sq_mul<NT, KS, STK>(Y, E);
        sq_each<NT>([&](int i, int n, int r) {
            E.t[i][n].re[r] = -G.t[i][n].im[r] - E.t[i][n].re[r];
            E.t[i][n].im[r] = G.t[i][n].re[r] - E.t[i][n].im[r];
        });
        return E;
    }
    int b = q - 2;   // the leading block
    const Sq<NT> Z = sq_mul<NT, KS, STK>(G, Y);
    block(p.tc[3 * b], p.tc[3 * b + 1], p.tc[3 * b + 2]);
    const double c3 = p.tc[3 * b + 3];
    sq_each<NT>([&](int i, int n, int r) {
        E.t[i][n].re[r] = fma(c3, Z.t[i][n].im[r], E.t[i][n].re[r]);
        E.t[i][n].im[r] = fma(-c3, Z.t[i][n].re[r], E.t[i][n].im[r]);
    });
    while (--b > 0) {
        const Sq<NT> W = sq_mul<NT, KS, STK>(Z, E);
        block(p.tc[3 * b], p.tc[3 * b + 1], p.tc[3 * b + 2]);
        sq_each<NT>([&](int i, int n, int r) {
            E.t[i][n].re[r] += W.t[i][n].im[r];
            E.t[i][n].im[r] -= W.t[i][n].re[r];
        });
    }
    // the last block: c0 left out, c1 = 1
    const Sq<NT> W = sq_mul<NT, KS, STK>(Z, E);
    const double c2 = p.tc[2];
    sq_each<NT>([&](int i, int n, int r) {
        E.t[i][n].re[r] = fma(-c2, Y.t[i][n].re[r], W.t[i][n].im[r]) - G.t[i][n].im[r];
        E.t[i][n].im[r] = fma(-c2, Y.t[i][n].im[r], G.t[i][n].re[r]) - W.t[i][n].re[r];
    });
    return E;
}

// exp(i G) - I by the degree-m Chebyshev series of cheb_parts on the interval
// [-theta, theta]: C + i P with C = sum e_i T_i(Y) and P = X sum b_i T_i(Y),
// X = G / theta, Y = 2 X^2 - I; `ec` the degree's row of even and odd
// coefficients.
template <int NT, int KS>
__device__ __forceinline__ Sq<NT> sq_cheb(const Sq<NT>& G, int m, double theta, const double* ec, const WLane& L) {
    const double inv = 1.0 / theta;
    const double* eb = ec + kChebHalf;
    const int qc = m / 2, qs = (m - 1) / 2;
    Sq<NT> X, C = sq_diagonal<NT>(L, ec[0]), Sp = sq_diagonal<NT>(L, eb[0]);
    sq_each<NT>([&](int i, int n, int r) {
        X.t[i][n].re[r] = G.t[i][n].re[r] * inv;
        X.t[i][n].im[r] = G.t[i][n].im[r] * inv;
    });
    auto add = [&](Sq<NT>& A, double c, const Sq<NT>& B) {
        sq_each<NT>([&](int i, int n, int r) {
            A.t[i][n].re[r] = fma(c, B.t[i][n].re[r], A.t[i][n].re[r]);
            A.t[i][n].im[r] = fma(c, B.t[i][n].im[r], A.t[i][n].im[r]);
        });
    };
    if (qc >= 1) {
        Sq<NT> Y = sq_mul<NT, KS>(X, X), Tm = sq_diagonal<NT>(L, 1.0);
        sq_each<NT>([&](int i, int n, int r) {
            Y.t[i][n].re[r] = fma(2.0, Y.t[i][n].re[r], -Tm.t[i][n].re[r]);
            Y.t[i][n].im[r] *= 2.0;
        });
        add(C, ec[1], Y);
        if (qs >= 1) add(Sp, eb[1], Y);
        Sq<NT> Tc = Y;
        for (int i = 2; i <= qc; ++i) {
            Sq<NT> Tn = sq_mul<NT, KS>(Y, Tc);
            sq_each<NT>([&](int a, int n, int r) {
                Tn.t[a][n].re[r] = fma(2.0, Tn.t[a][n].re[r], -Tm.t[a][n].re[r]);
                Tn.t[a][n].im[r] = fma(2.0, Tn.t[a][n].im[r], -Tm.t[a][n].im[r]);
            });
            add(C, ec[i], Tn);
            if (i <= qs) add(Sp, eb[i], Tn);
            Tm = Tc;
            Tc = Tn;
        }
    }
    Sq<NT> P;
    if (qs >= 1) {
        P = sq_mul<NT, KS>(X, Sp);
    } else {
        sq_each<NT>([&](int i, int n, int r) {
            P.t[i][n].re[r] = eb[0] * X.t[i][n].re[r];
            P.t[i][n].im[r] = eb[0] * X.t[i][n].im[r];
        });
    }
    sq_each<NT>([&](int i, int n, int r) {
        C.t[i][n].re[r] = (C.t[i][n].re[r] - (sq_diag(L, i, n, r) ? 1.0 : 0.0)) - P.t[i][n].im[r];
        C.t[i][n].im[r] += P.t[i][n].re[r];
    });
    return C;
}

typedef double d2_t __attribute__((ext_vector_type(2)));

// Order this wave's LDS writes before its reads of other lanes' entries (and
// the reverse).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The adjoint of a matrix, tile by tile through a 16 x 17 scratch tile of the
// wave (row stride 17 entries: rows and columns both read without conflicts).
constexpr int kScratchTile = 16 * 17;   // d2_t entries
template <int NT>
__device__ __forceinline__ Sq<NT> sq_adjoint(const Sq<NT>& X, d2_t* scr, const WLane& L) {
    Sq<NT> o;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            wave_lds_fence();
#pragma unroll
            for (int r = 0; r < 4; ++r)
                scr[(L.g + 4 * r) * 17 + L.j] = d2_t{X.t[n][i].re[r], X.t[n][i].im[r]};
            wave_lds_fence();
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const d2_t v = scr[L.j * 17 + L.g + 4 * r];
                o.t[i][n].re[r] = v.x;
                o.t[i][n].im[r] = -v.y;
            }
        }
    return o;
}

// [X, Y] = X Y - (X Y)^H of Hermitian X, Y.
template <int NT, int KS>
__device__ __forceinline__ Sq<NT> sq_commutator(const Sq<NT>& X, const Sq<NT>& Y, d2_t* scr, const WLane& L) {
    Sq<NT> Z = sq_mul<NT, KS>(X, Y);
    const Sq<NT> A = sq_adjoint<NT>(Z, scr, L);
    sq_each<NT>([&](int i, int n, int r) {
        Z.t[i][n].re[r] -= A.t[i][n].re[r];
        Z.t[i][n].im[r] -= A.t[i][n].im[r];
    });
    return Z;
}

// E <- (I + E)^2 - I = 2 E + E E, s times.
template <int NT, int KS>
__device__ __forceinline__ void sq_square(Sq<NT>& E, int s, d2_t* scr, const WLane& L) {
    for (int q = 0; q < s; ++q) {
        const Sq<NT> P = sq_mul<NT, KS>(sq_adjoint<NT>(E, scr, L), E);
        sq_each<NT>([&](int i, int n, int r) {
            E.t[i][n].re[r] = fma(2.0, E.t[i][n].re[r], P.t[i][n].re[r]);
            E.t[i][n].im[r] = fma(2.0, E.t[i][n].im[r], P.t[i][n].im[r]);
        });
    }
}

// ||G||_1 (bound) of the Hermitian G as its largest row sum.
template <int NT>
__device__ __forceinline__ double sq_norm1(const Sq<NT>& G) {
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float s = 0.0f;
#pragma unroll
            for (int n = 0; n < NT; ++n) s += abs_bound_f(G.t[i][n].re[r], G.t[i][n].im[r]);
            m = fmaxf(m, row16_sum_f(s));
        }
    return rows_max_f(m);
}

// Node (chain or tree product) in memory: [D][D] complex128, row-major.
template <int NT>
__device__ __forceinline__ void sq_node_store(double* node, const Sq<NT>& Q, const WLane& L) {
    d2_t* o = reinterpret_cast<d2_t*>(node);
    sq_each<NT>([&](int i, int n, int r) {
        o[(16 * i + L.g + 4 * r) * (16 * NT) + 16 * n + L.j] = d2_t{Q.t[i][n].re[r], Q.t[i][n].im[r]};
    });
}

// Nodes shared inside the launch travel as agent-scope atomic accesses
// (node_store_coherent: why no fences are needed).
template <int NT>
__device__ __forceinline__ void sq_node_publish(double* node, const Sq<NT>& Q, const WLane& L) {
    sq_each<NT>([&](int i, int n, int r) {
        double* o = node + ((16 * i + L.g + 4 * r) * (16 * NT) + 16 * n + L.j) * 2;
        __hip_atomic_store(o, Q.t[i][n].re[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(o + 1, Q.t[i][n].im[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// A published node, or with ADJ its adjoint (the left factor of a product).
template <int NT, bool ADJ>
__device__ __forceinline__ Sq<NT> sq_node_fetch(double* node, const WLane& L) {
    Sq<NT> Q;
    sq_each<NT>([&](int i, int n, int r) {
        const int row = 16 * i + L.g + 4 * r, col = 16 * n + L.j;
        double* o = node + (ADJ ? col * (16 * NT) + row : row * (16 * NT) + col) * 2;
        Q.t[i][n].re[r] = __hip_atomic_load(o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        Q.t[i][n].im[r] = __hip_atomic_load(o + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ADJ) Q.t[i][n].im[r] = -Q.t[i][n].im[r];
    });
    return Q;
}

// Root product into U_out.
template <int NT>
__device__ __forceinline__ void sq_store_root(const PropParams& p, const Sq<NT>& Q, const WLane& L) {
    sq_each<NT>([&](int i, int n, int r) {
        const int row = 16 * i + L.g + 4 * r, col = 16 * n + L.j;
        if (row < p.du && col < p.du) {
            p.U_out[(row * p.du + col) * 2 + 0] = Q.t[i][n].re[r];
            p.U_out[(row * p.du + col) * 2 + 1] = Q.t[i][n].im[r];
        }
    });
}

// Product of consecutive teams' matrices, team 0 the earliest: teams 1 and 3
// hand theirs to 0 and 2 through LDS, then 2 to 0 (later on the left).  Teams
// from `live` on hold nothing.  The block's four waves all call it.  slots:
// four of D (D + 1) entries; the handed matrix is written by rows and read as
// its adjoint, both without bank conflicts.
constexpr int kWaveTeams = 4;
template <int NT>
constexpr int sq_slot_entries() { return 16 * NT * (16 * NT + 1); }

template <int NT, int KS>
__device__ __forceinline__ void sq_combine(Sq<NT>& Q, int team, int live, d2_t* slots, const WLane& L) {
    constexpr int LD = 16 * NT + 1;
    d2_t* own = slots + team * sq_slot_entries<NT>();
#pragma unroll
    for (int st = 1; st < kWaveTeams; st <<= 1) {
        __syncthreads();
        if ((team & (2 * st - 1)) == st && team < live)
            sq_each<NT>([&](int i, int n, int r) {
                own[(16 * i + L.g + 4 * r) * LD + 16 * n + L.j] = d2_t{Q.t[i][n].re[r], Q.t[i][n].im[r]};
            });
        __syncthreads();
        if ((team & (2 * st - 1)) == 0 && team + st < live) {
            const d2_t* later = slots + (team + st) * sq_slot_entries<NT>();
            Sq<NT> S;
            sq_each<NT>([&](int i, int n, int r) {
                const d2_t v = later[(16 * n + L.j) * LD + 16 * i + L.g + 4 * r];
                S.t[i][n].re[r] = v.x;
                S.t[i][n].im[r] = -v.y;
            });
            Q = sq_mul<NT, KS>(S, Q);
        }
    }
}

// The ticketed product tree (fan-in kFanIn) of blocks of four one-wave teams,
// which stay together into it: team 0 publishes the block's node and takes
// its group's ticket; in the group's last arrival team w multiplies nodes
// 2 w + 1 and 2 w, read straight from memory, and sq_combine does the rest:
// three dependent products per level.
template <int NT, int KS>
__device__ void sq_tree(const PropParams& p, int64_t leaf, Sq<NT>& Q, int team, d2_t* slots, int* tick,
                        const WLane& L) {
    static_assert(2 * kWaveTeams == kFanIn, "two nodes per team");
    constexpr int64_t NN = (int64_t)256 * NT * NT * 2;
    int64_t idx = leaf, cnt = p.n_leaves, off = 0;
    while (cnt > 1) {
        const int64_t pcnt = (cnt + kFanIn - 1) / kFanIn, poff = off + cnt, grp = idx / kFanIn;
        const int64_t first = grp * kFanIn;
        const int members = (int)(min(cnt, first + kFanIn) - first);
        if (members == 1) {
            if (p.store_nodes && team == 0) sq_node_store<NT>(p.nodes + (off + idx) * NN, Q, L);
        } else {
            if (team == 0) {
                sq_node_publish<NT>(p.nodes + (off + idx) * NN, Q, L);
                unsigned v = 0;
                if (L.lane == 0) v = atomicAdd(&p.counters[poff + grp], 1u);
                const unsigned t = (unsigned)__builtin_amdgcn_readfirstlane((int)v);
                if (t == (unsigned)(members - 1) && L.lane == 0) atomicExch(&p.counters[poff + grp], 0u);
                if (L.lane == 0) *tick = (int)t;
            }
            __syncthreads();
            const int t = *tick;
            __syncthreads();
            if (t != members - 1) return;   // the whole block leaves
            double* nd = p.nodes + (off + first + 2 * team) * NN;
            if (2 * team + 1 < members) {
                const Sq<NT> S = sq_node_fetch<NT, true>(nd + NN, L);
                Q = sq_mul<NT, KS>(S, sq_node_fetch<NT, false>(nd, L));
            } else if (2 * team < members) {
                Q = sq_node_fetch<NT, false>(nd, L);
            }
            sq_combine<NT, KS>(Q, team, (members + 1) / 2, slots, L);
        }
        idx = grp;
        off = poff;
        cnt = pcnt;
    }
    if (team != 0) return;
    if (p.store_nodes) sq_node_store<NT>(p.nodes + off * NN, Q, L);
    sq_store_root<NT>(p, Q, L);
}

}  // namespace
}  // namespace pm
