// One-wave teams: the FP64 MFMA engine of dimensions up to 32.
//
// One wave carries a chain and holds every matrix in registers, in the
// accumulator layout of v_mfma_f64_16x16x4f64 (lane 16 g + j holds rows
// g + 4 r, r = 0..3, of column j of a 16 x 16 tile).  Register r of tile (k, n)
// is the B operand of a k-slice as it stands, and register r of tile (k, i) of
// S the A operand of S^H: a product S^H X takes both operands from the lane's
// own registers.  So the engine computes S^H X only: S X for the Hermitian
// factors of the series, and for the chain it carries E = exp(i G) - I, whose
// adjoint is exp(-i G) - I: Q <- Q + E^H Q.  No product touches LDS and no wave
// waits for another one.
//
// Shapes (a lane's entries of a matrix are numbered e = 0 .. kRegs - 1):
//   Wide<NT, KS>  one 16 NT x 16 NT matrix, NT x NT tiles; KS the k-slices (of
//                 four rows) that the embedded dimension reaches, du <= 4 KS
//                 (rows and columns past them are zero in every product);
//   Pair<KS>      two matrices of dimension <= 4 KS <= 8 that advance together,
//                 in the diagonal 8 x 8 blocks of one tile: lanes j < 8 hold the
//                 first, lanes j >= 8 the second, rows g + 4 e of column j & 7.
//                 Their products are one stacked product [A_a; A_b] [B_a, B_b]
//                 with K = 4 KS, of which each lane keeps its own block's rows.
#pragma once

#include "mfma_tiles.h"

namespace pm {
namespace {

struct WLane {
    int lane, g, j;
};

template <int NT_, int KS_>
struct Wide {
    static constexpr int NT = NT_, KS = KS_, RT = (KS + 3) / 4;
    static constexpr bool kPair = false;
    static constexpr int kRegs = 4 * NT * NT;
    static constexpr int at(int i, int n, int r) { return (i * NT + n) * 4 + r; }
    static __device__ __forceinline__ int row(const WLane& L, int e) { return 16 * (e / (4 * NT)) + L.g + 4 * (e & 3); }
    static __device__ __forceinline__ int col(const WLane& L, int e) { return 16 * (e / 4 % NT) + L.j; }
};

template <int KS_>
struct Pair {
    static_assert(KS_ <= 2, "blocks of 8 x 8");
    static constexpr int NT = 1, KS = KS_;
    static constexpr bool kPair = true;
    static constexpr int kRegs = KS;
    static __device__ __forceinline__ int row(const WLane& L, int e) { return L.g + 4 * e; }
    static __device__ __forceinline__ int col(const WLane& L, int) { return L.j & 7; }
};

// A lane's entries of a matrix (of two matrices for Pair).
template <class S>
struct Mx {
    double re[S::kRegs], im[S::kRegs];
};

template <class S, class F>
__device__ __forceinline__ void mx_each(F f) {
#pragma unroll
    for (int e = 0; e < S::kRegs; ++e) f(e);
}

template <class S>
__device__ __forceinline__ bool mx_diag(const WLane& L, int e) { return S::row(L, e) == S::col(L, e); }

template <class S>
__device__ __forceinline__ Mx<S> mx_diagonal(const WLane& L, double v) {
    Mx<S> m;
    mx_each<S>([&](int e) {
        m.re[e] = mx_diag<S>(L, e) ? v : 0.0;
        m.im[e] = 0.0;
    });
    return m;
}

template <class S>
__device__ __forceinline__ void mx_add(Mx<S>& y, const Mx<S>& x) {
    mx_each<S>([&](int e) {
        y.re[e] += x.re[e];
        y.im[e] += x.im[e];
    });
}

// A^H X as three real products chained through the accumulator:
// k = (Ar - Ai) Xr, Re = k + Ai (Xr + Xi), Im = k + Ar (Xi - Xr).  Re and Im
// start from k as their MFMAs' C operand, so no sums follow the matrix
// instructions (the usual t1 + t2, t3 - t1 + t2 take 12 more vector
// instructions a tile, and none of those overlaps an FP64 MFMA of its SIMD).
// The operands' sums come ahead of the MFMAs: one right before the MFMA that
// reads it would cost wait states each time.
template <class S>
__device__ __forceinline__ Mx<S> mx_mul(const Mx<S>& A, const Mx<S>& X) {
    Mx<S> out;
    constexpr int KS = S::KS;
    if constexpr (S::kPair) {
        double sd[KS], xp[KS], xm[KS];
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            sd[q] = A.re[q] - A.im[q];
            xp[q] = X.re[q] + X.im[q];
            xm[q] = X.im[q] - X.re[q];
        }
        __builtin_amdgcn_sched_barrier(0);
        d4_t kk = {0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < KS; ++q) kk = mfma16(sd[q], X.re[q], kk);
        d4_t re = kk, im = kk;
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            re = mfma16(A.im[q], xp[q], re);
            im = mfma16(A.re[q], xm[q], im);
        }
        __builtin_amdgcn_sched_barrier(0);
        // rows of the lane's own block (the others hold cross products)
        const bool hi = (__lane_id() & 8) != 0;
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            out.re[q] = hi ? re[q + 2] : re[q];
            out.im[q] = hi ? im[q + 2] : im[q];
        }
    } else {
        constexpr int NT = S::NT, RT = S::RT;
        double sd[RT][KS];
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int q = 0; q < KS; ++q) {
                const int e = S::at(q >> 2, i, q & 3);
                sd[i][q] = A.re[e] - A.im[e];
            }
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            double xp[KS], xm[KS];
#pragma unroll
            for (int q = 0; q < KS; ++q) {
                const int e = S::at(q >> 2, n, q & 3);
                xp[q] = X.re[e] + X.im[e];
                xm[q] = X.im[e] - X.re[e];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                d4_t kk = {0, 0, 0, 0};
                if (i < RT && n < RT) {
#pragma unroll
                    for (int q = 0; q < KS; ++q) kk = mfma16(sd[i][q], X.re[S::at(q >> 2, n, q & 3)], kk);
                }
                d4_t re = kk, im = kk;
                if (i < RT && n < RT) {
#pragma unroll
                    for (int q = 0; q < KS; ++q) {
                        const int e = S::at(q >> 2, i, q & 3);
                        re = mfma16(A.im[e], xp[q], re);
                        im = mfma16(A.re[e], xm[q], im);
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    out.re[S::at(i, n, r)] = re[r];
                    out.im[S::at(i, n, r)] = im[r];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return out;
}

// X + A^H X.
template <class S>
__device__ __forceinline__ Mx<S> mx_apply(const Mx<S>& A, const Mx<S>& X) {
    Mx<S> y = mx_mul<S>(A, X);
    mx_add<S>(y, X);
    return y;
}

// A^H X of unitary A (a chain's or a node's adjoint) as X + (A - I)^H X: the
// product rounds relative to ||A - I||, which is small where chains are short and
// the tree takes over their products (a full product rounds ten times as much).
// 27 levels, 278 slices: gradient 1.1e-14 -> 4.0e-15, U(T) 8.0e-15 -> 1.5e-15; 8 levels,
// 1000 slices of a trajectory 6.2e-15 -> 2.5e-15 (16 levels, 1000 slices 22.1 -> 22.3 us).
template <class S>
__device__ __forceinline__ Mx<S> mx_join(Mx<S> A, const Mx<S>& X, const WLane& L) {
    mx_each<S>([&](int e) { A.re[e] -= mx_diag<S>(L, e) ? 1.0 : 0.0; });
    return mx_apply<S>(A, X);
}

// exp(i G) - I for the (pre-scaled) Hermitian G by evaluation scheme q
// (scheme_degree(q); coefficients p.tc[k] = 1/k!, zero past the degree cap),
// Paterson-Stockmeyer in blocks of three powers with Y = G G, Z = G Y:
//   q = 0  i G;   q = 1  i G - Y/2;   q = 2  i G - Y (1/2 + i G/6 - Y/24);
//   q >= 3 blocks B_i = c_{3i} + c_{3i+1} i G - c_{3i+2} Y over powers of
//          (i G)^3 = -i Z, X <- B_i - i Z X: q products in all.
// Every left factor is Hermitian.
template <class S>
__device__ __forceinline__ Mx<S> mx_expm1(const PropParams& p, const Mx<S>& G, int q, const WLane& L) {
    Mx<S> E;
    if (q == 0) {
        mx_each<S>([&](int e) {
            E.re[e] = -G.im[e];
            E.im[e] = G.re[e];
        });
        return E;
    }
    const Mx<S> Y = mx_mul<S>(G, G);
    // c0 I + c1 i G - c2 Y into E
    auto block = [&](double c0, double c1, double c2) {
        mx_each<S>([&](int e) {
            E.re[e] = fma(-c1, G.im[e], fma(-c2, Y.re[e], mx_diag<S>(L, e) ? c0 : 0.0));
            E.im[e] = fma(c1, G.re[e], -c2 * Y.im[e]);
        });
    };
    if (q <= 2) {
        if (q == 1) {
            block(0.0, 1.0, p.tc[2]);
            return E;
        }
        block(p.tc[2], p.tc[3], p.tc[4]);
        E = mx_mul<S>(Y, E);
        mx_each<S>([&](int e) {
            E.re[e] = -G.im[e] - E.re[e];
            E.im[e] = G.re[e] - E.im[e];
        });
        return E;
    }
    int b = q - 2;   // the leading block
    const Mx<S> Z = mx_mul<S>(G, Y);
    block(p.tc[3 * b], p.tc[3 * b + 1], p.tc[3 * b + 2]);
    const double c3 = p.tc[3 * b + 3];
    mx_each<S>([&](int e) {
        E.re[e] = fma(c3, Z.im[e], E.re[e]);
        E.im[e] = fma(-c3, Z.re[e], E.im[e]);
    });
    while (--b > 0) {
        const Mx<S> W = mx_mul<S>(Z, E);
        block(p.tc[3 * b], p.tc[3 * b + 1], p.tc[3 * b + 2]);
        mx_each<S>([&](int e) {
            E.re[e] += W.im[e];
            E.im[e] -= W.re[e];
        });
    }
    // the last block: c0 left out, c1 = 1
    const Mx<S> W = mx_mul<S>(Z, E);
    const double c2 = p.tc[2];
    mx_each<S>([&](int e) {
        E.re[e] = fma(-c2, Y.re[e], W.im[e]) - G.im[e];
        E.im[e] = fma(-c2, Y.im[e], G.re[e]) - W.re[e];
    });
    return E;
}

typedef double d2_t __attribute__((ext_vector_type(2)));

// A matrix put aside in LDS, the lane's entries as they are, and taken back.  (The
// compiler must not carry them over in registers after all.)
template <class S>
constexpr int mx_aside_entries() { return 64 * S::kRegs; }
template <class S>
__device__ __forceinline__ void mx_put_aside(d2_t* to, const Mx<S>& X, const WLane& L) {
    mx_each<S>([&](int e) { to[e * 64 + L.lane] = d2_t{X.re[e], X.im[e]}; });
    asm volatile("" ::: "memory");
}
template <class S>
__device__ __forceinline__ void mx_take_back(Mx<S>& X, const d2_t* from, const WLane& L) {
    mx_each<S>([&](int e) {
        const d2_t v = from[e * 64 + L.lane];
        X.re[e] = v.x;
        X.im[e] = v.y;
    });
}

// exp(i G) - I by the degree-m Chebyshev series on the interval
// [-theta, theta], the spectrum's bound (eq. chebychev_series with
// alpha = -theta, beta = theta), split into its even and odd halves.  With
// X = G / theta and Y = T_2(X) = 2 X^2 - I, T_2j(X) = T_j(Y) and
// T_{2j+1}(X) = X (2 sum_{i=1..j} (-1)^{j-i} T_i(Y) + (-1)^j I), so
//   exp(i G) = C + i P,  C = sum_{i <= m/2} e_i T_i(Y),
//   P = X sum_{i <= (m-1)/2} b_i T_i(Y),
// e_0 = J_0, e_i = 2 (-1)^i J_2i, and b the alternating suffix sums of the
// odd coefficients (`ec`: the degree's row of e, then of b, kChebHalf each).
// floor(m/2) + 1 products, all with a Hermitian left factor, where the
// Clenshaw recurrence in X takes m.  Two tiles wide X waits in LDS (`aside`):
// besides it the series holds six matrices of 64 registers.
template <class S>
__device__ __forceinline__ Mx<S> mx_cheb(const Mx<S>& G, int m, double theta, const double* ec, d2_t* aside,
                                         const WLane& L) {
    const double inv = 1.0 / theta;
    const double* eb = ec + kChebHalf;
    const int qc = m / 2, qs = (m - 1) / 2;
    Mx<S> X, C = mx_diagonal<S>(L, ec[0]), Sp = mx_diagonal<S>(L, eb[0]);
    mx_each<S>([&](int e) {
        X.re[e] = G.re[e] * inv;
        X.im[e] = G.im[e] * inv;
    });
    auto add = [&](Mx<S>& A, double c, const Mx<S>& B) {
        mx_each<S>([&](int e) {
            A.re[e] = fma(c, B.re[e], A.re[e]);
            A.im[e] = fma(c, B.im[e], A.im[e]);
        });
    };
    if constexpr (S::NT > 1) mx_put_aside<S>(aside, X, L);
    if (qc >= 1) {
        Mx<S> Y = mx_mul<S>(X, X), Tm = mx_diagonal<S>(L, 1.0);
        mx_each<S>([&](int e) {
            Y.re[e] = fma(2.0, Y.re[e], -Tm.re[e]);
            Y.im[e] *= 2.0;
        });
        add(C, ec[1], Y);
        if (qs >= 1) add(Sp, eb[1], Y);
        // T_i over T_{i-2}, in turns (no copies, no third matrix)
        auto next = [&](int i, const Mx<S>& Tc, Mx<S>& Tn) {
            const Mx<S> Z = mx_mul<S>(Y, Tc);
            mx_each<S>([&](int e) {
                Tn.re[e] = fma(2.0, Z.re[e], -Tn.re[e]);
                Tn.im[e] = fma(2.0, Z.im[e], -Tn.im[e]);
            });
            add(C, ec[i], Tn);
            if (i <= qs) add(Sp, eb[i], Tn);
        };
        Mx<S> Tc = Y;
        for (int i = 2; i <= qc; i += 2) {
            next(i, Tc, Tm);
            if (i == qc) break;
            next(i + 1, Tm, Tc);
        }
    }
    Mx<S> P;
    if constexpr (S::NT > 1) mx_take_back<S>(X, aside, L);
    if (qs >= 1) {
        P = mx_mul<S>(X, Sp);
    } else {
        mx_each<S>([&](int e) {
            P.re[e] = eb[0] * X.re[e];
            P.im[e] = eb[0] * X.im[e];
        });
    }
    mx_each<S>([&](int e) {
        C.re[e] = (C.re[e] - (mx_diag<S>(L, e) ? 1.0 : 0.0)) - P.im[e];
        C.im[e] += P.re[e];
    });
    return C;
}

// Order this wave's LDS writes before its reads of other lanes' entries (and
// the reverse).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The adjoint of a matrix through the wave's scratch tile: tiles one by one
// with a row stride of 17 entries (8 x 8 blocks: 9), so that rows and columns
// are both accessed without conflicts.
constexpr int kScratchTile = 16 * 17;   // d2_t entries
template <class S>
__device__ __forceinline__ Mx<S> mx_adjoint(const Mx<S>& X, d2_t* scr, const WLane& L) {
    Mx<S> o;
    if constexpr (S::kPair) {
        d2_t* b = scr + (L.j >> 3) * 72;
        const int c = L.j & 7;
        wave_lds_fence();
        mx_each<S>([&](int e) { b[(L.g + 4 * e) * 9 + c] = d2_t{X.re[e], X.im[e]}; });
        wave_lds_fence();
        mx_each<S>([&](int e) {
            // (with KS = 1 nothing was written to rows 4 and on)
            const d2_t v = b[(S::KS == 1 ? c & 3 : c) * 9 + L.g + 4 * e];
            const bool in = S::KS > 1 || c < 4;
            o.re[e] = in ? v.x : 0.0;
            o.im[e] = in ? -v.y : 0.0;
        });
    } else {
#pragma unroll
        for (int i = 0; i < S::NT; ++i)
#pragma unroll
            for (int n = 0; n < S::NT; ++n) {
                wave_lds_fence();
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    scr[(L.g + 4 * r) * 17 + L.j] = d2_t{X.re[S::at(n, i, r)], X.im[S::at(n, i, r)]};
                wave_lds_fence();
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const d2_t v = scr[L.j * 17 + L.g + 4 * r];
                    o.re[S::at(i, n, r)] = v.x;
                    o.im[S::at(i, n, r)] = -v.y;
                }
            }
    }
    return o;
}

// [X, Y] = X Y - (X Y)^H of Hermitian X, Y.
template <class S>
__device__ __forceinline__ Mx<S> mx_commutator(const Mx<S>& X, const Mx<S>& Y, d2_t* scr, const WLane& L) {
    Mx<S> Z = mx_mul<S>(X, Y);
    const Mx<S> A = mx_adjoint<S>(Z, scr, L);
    mx_each<S>([&](int e) {
        Z.re[e] -= A.re[e];
        Z.im[e] -= A.im[e];
    });
    return Z;
}

// E <- (I + E)^2 - I = 2 E + E E, s times.
template <class S>
__device__ __forceinline__ void mx_square(Mx<S>& E, int s, d2_t* scr, const WLane& L) {
    for (int q = 0; q < s; ++q) {
        const Mx<S> P = mx_mul<S>(mx_adjoint<S>(E, scr, L), E);
        mx_each<S>([&](int e) {
            E.re[e] = fma(2.0, E.re[e], P.re[e]);
            E.im[e] = fma(2.0, E.im[e], P.im[e]);
        });
    }
}

// ||G||_1 (bound) of the Hermitian G as its largest row sum (Pair: over both).
template <class S>
__device__ __forceinline__ double mx_norm1(const Mx<S>& G) {
    float m = 0.0f;
    if constexpr (S::kPair) {
        mx_each<S>([&](int e) {
            float s = abs_bound_f(G.re[e], G.im[e]);
            s += __shfl_xor(s, 1);
            s += __shfl_xor(s, 2);
            s += __shfl_xor(s, 4);
            m = fmaxf(m, fmaxf(s, __shfl_xor(s, 8)));
        });
    } else {
#pragma unroll
        for (int i = 0; i < S::NT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float s = 0.0f;
#pragma unroll
                for (int n = 0; n < S::NT; ++n) s += abs_bound_f(G.re[S::at(i, n, r)], G.im[S::at(i, n, r)]);
                m = fmaxf(m, row16_sum_f(s));
            }
    }
    return rows_max_f(m);
}

// Node (chain or tree product) in memory: [D][D] complex128, row-major.
template <class S>
__device__ __forceinline__ void mx_node_store(double* node, const Mx<S>& Q, const WLane& L) {
    d2_t* o = reinterpret_cast<d2_t*>(node);
    mx_each<S>([&](int e) { o[S::row(L, e) * (16 * S::NT) + S::col(L, e)] = d2_t{Q.re[e], Q.im[e]}; });
}

// A node of an earlier launch, or with ADJ its adjoint (a left factor).
template <class S, bool ADJ>
__device__ __forceinline__ Mx<S> mx_node_load(const double* node, const WLane& L) {
    const d2_t* o = reinterpret_cast<const d2_t*>(node);
    Mx<S> Q;
    mx_each<S>([&](int e) {
        const d2_t v = o[ADJ ? S::col(L, e) * (16 * S::NT) + S::row(L, e) : S::row(L, e) * (16 * S::NT) + S::col(L, e)];
        Q.re[e] = v.x;
        Q.im[e] = ADJ ? -v.y : v.y;
    });
    return Q;
}

// Nodes shared inside the launch are read as agent-scope atomic accesses
// (node_store_coherent: why no fences are needed).
template <class S, bool ADJ>
__device__ __forceinline__ Mx<S> mx_node_fetch(double* node, const WLane& L) {
    Mx<S> Q;
    mx_each<S>([&](int e) {
        const int row = S::row(L, e), col = S::col(L, e);
        double* o = node + (ADJ ? col * (16 * S::NT) + row : row * (16 * S::NT) + col) * 2;
        Q.re[e] = __hip_atomic_load(o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        Q.im[e] = __hip_atomic_load(o + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ADJ) Q.im[e] = -Q.im[e];
    });
    return Q;
}

constexpr int kWaveTeams = 4;
template <class S>
constexpr int mx_slot_entries() { return 16 * S::NT * (16 * S::NT + 1); }

// A block's product as its waves hold it: one tile wide the whole of it in team 0,
// two wide a tile in each team.
template <class S>
struct Part {
    static_assert(S::NT == 1 || S::NT * S::NT == kWaveTeams, "a tile per team");
    double re[4], im[4];
    static __device__ __forceinline__ bool mine(int team) { return S::NT > 1 || team == 0; }
    static __device__ __forceinline__ int row(const WLane& L, int team, int r) { return 16 * (S::NT > 1 ? team >> 1 : 0) + L.g + 4 * r; }
    static __device__ __forceinline__ int col(const WLane& L, int team) { return 16 * (S::NT > 1 ? team & 1 : 0) + L.j; }
};

template <class S>
__device__ __forceinline__ void part_store(double* node, const Part<S>& Q, int team, const WLane& L) {
    d2_t* o = reinterpret_cast<d2_t*>(node);
#pragma unroll
    for (int r = 0; r < 4; ++r) o[Q.row(L, team, r) * (16 * S::NT) + Q.col(L, team)] = d2_t{Q.re[r], Q.im[r]};
}

// Agent-scope atomic stores, complete when this returns.
template <class S>
__device__ __forceinline__ void part_publish(double* node, const Part<S>& Q, int team, const WLane& L) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        double* o = node + (Q.row(L, team, r) * (16 * S::NT) + Q.col(L, team)) * 2;
        __hip_atomic_store(o, Q.re[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(o + 1, Q.im[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Root product into U_out.
template <class S>
__device__ __forceinline__ void part_store_root(const PropParams& p, const Part<S>& Q, int team, const WLane& L) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = Q.row(L, team, r), col = Q.col(L, team);
        if (row < p.du && col < p.du) {
            p.U_out[(row * p.du + col) * 2 + 0] = Q.re[r];
            p.U_out[(row * p.du + col) * 2 + 1] = Q.im[r];
        }
    }
}

// Tiles (i0, n) .. (i0 + NI - 1, n) of A X = X + (A - I) X (mx_join) for two
// matrices in handover slots.
template <class S, int NI>
__device__ __forceinline__ void mx_slot_tiles(const d2_t* a, const d2_t* x, int i0, int n, Part<S> (&out)[NI],
                                              const WLane& L) {
    constexpr int LD = 16 * S::NT + 1, KS = S::KS;
    double xr[KS], xp[KS], xm[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) {
        const d2_t v = x[(16 * (q >> 2) + L.g + 4 * (q & 3)) * LD + 16 * n + L.j];
        xr[q] = v.x;
        xp[q] = v.x + v.y;
        xm[q] = v.y - v.x;
    }
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        const int i = i0 + t;
        double ar[KS], ai[KS], sd[KS];
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            const int row = 16 * (q >> 2) + L.g + 4 * (q & 3), col = 16 * i + L.j;
            const d2_t v = a[col * LD + row];
            ar[q] = v.x - (row == col ? 1.0 : 0.0);
            ai[q] = -v.y;
            sd[q] = ar[q] - ai[q];
        }
        d4_t kk = {0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < KS; ++q) kk = mfma16(sd[q], xr[q], kk);
        d4_t re = kk, im = kk;
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            re = mfma16(ai[q], xp[q], re);
            im = mfma16(ar[q], xm[q], im);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const d2_t v = x[(16 * i + L.g + 4 * r) * LD + 16 * n + L.j];
            out[t].re[r] = re[r] + v.x;
            out[t].im[r] = im[r] + v.y;
        }
    }
}

// Product of consecutive teams' matrices, team 0 the earliest (later on the left);
// teams from `live` on hold nothing.  The block's four waves all call it.  slots:
// four of D (D + 1) entries; a matrix is written by rows and read as its adjoint,
// both without bank conflicts.
// One tile wide, teams 1 and 3 hand theirs to 0 and 2, then 2 to 0.  Two tiles wide
// a product takes one wave 2.6 us, so the idle ones share it: two waves a product
// (a column of tiles each), then four (a tile each).  27 levels, 100 slices 59.7 ->
// 49.5 us (a handover and two levels of the tree), 1000 slices 80.0 -> 65.6 us.
template <class S>
__device__ __forceinline__ Part<S> mx_combine(Mx<S>& Q, int team, int live, d2_t* slots, const WLane& L) {
    constexpr int LD = 16 * S::NT + 1;
    d2_t* own = slots + team * mx_slot_entries<S>();
    auto hand = [&]() { mx_each<S>([&](int e) { own[S::row(L, e) * LD + S::col(L, e)] = d2_t{Q.re[e], Q.im[e]}; }); };
    Part<S> P;
    if constexpr (S::NT == 1) {
#pragma unroll
        for (int st = 1; st < kWaveTeams; st <<= 1) {
            __syncthreads();
            if ((team & (2 * st - 1)) == st && team < live) hand();
            __syncthreads();
            if ((team & (2 * st - 1)) == 0 && team + st < live) {
                const d2_t* later = slots + (team + st) * mx_slot_entries<S>();
                Mx<S> A;
                mx_each<S>([&](int e) {
                    const d2_t v = later[S::col(L, e) * LD + S::row(L, e)];
                    A.re[e] = v.x;
                    A.im[e] = -v.y;
                });
                Q = mx_join<S>(A, Q, L);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            P.re[r] = Q.re[r];
            P.im[r] = Q.im[r];
        }
    } else {
        constexpr int SE = mx_slot_entries<S>();
        __syncthreads();
        if (team < live) hand();
        __syncthreads();
        if (live > 2) {
            const int pair = team & 2, n = team & 1;
            Part<S> C[2];
            if (pair + 1 < live) mx_slot_tiles<S, 2>(slots + (pair + 1) * SE, slots + pair * SE, 0, n, C, L);
            __syncthreads();
            if (pair + 1 < live)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        slots[pair * SE + (16 * i + L.g + 4 * r) * LD + 16 * n + L.j] = d2_t{C[i].re[r], C[i].im[r]};
            __syncthreads();
        }
        if (live > 1) {
            Part<S> C[1];
            mx_slot_tiles<S, 1>(slots + (live > 2 ? 2 : 1) * SE, slots, team >> 1, team & 1, C, L);
            P = C[0];
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const d2_t v = slots[P.row(L, team, r) * LD + P.col(L, team)];
                P.re[r] = v.x;
                P.im[r] = v.y;
            }
        }
    }
    return P;
}

// The ticketed product tree (fan-in kFanIn) of blocks of four one-wave teams,
// which stay together into it: the block's node is published and team 0 takes its
// group's ticket; in the group's last arrival team w multiplies nodes 2 w + 1 and
// 2 w, read straight from memory, and mx_combine does the rest.
template <class S>
__device__ void mx_tree(const PropParams& p, int64_t leaf, Part<S> Q, int team, d2_t* slots, int* tick,
                        const WLane& L) {
    static_assert(2 * kWaveTeams == kFanIn && !S::kPair, "two nodes per team");
    constexpr int64_t NN = (int64_t)256 * S::NT * S::NT * 2;
    const bool mine = Q.mine(team);
    int64_t idx = leaf, cnt = p.n_leaves, off = 0;
    while (cnt > 1) {
        const int64_t pcnt = (cnt + kFanIn - 1) / kFanIn, poff = off + cnt, grp = idx / kFanIn;
        const int64_t first = grp * kFanIn;
        const int members = (int)(min(cnt, first + kFanIn) - first);
        if (members == 1) {
            if (p.store_nodes && mine) part_store<S>(p.nodes + (off + idx) * NN, Q, team, L);
        } else {
            if (mine) part_publish<S>(p.nodes + (off + idx) * NN, Q, team, L);
            if constexpr (S::NT > 1) __syncthreads();   // every team's tile is out
            if (team == 0) {
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
            Mx<S> M;
            if (2 * team + 1 < members) {
                const Mx<S> A = mx_node_fetch<S, true>(nd + NN, L);
                M = mx_join<S>(A, mx_node_fetch<S, false>(nd, L), L);
            } else if (2 * team < members) {
                M = mx_node_fetch<S, false>(nd, L);
            }
            Q = mx_combine<S>(M, team, (members + 1) / 2, slots, L);
        }
        idx = grp;
        off = poff;
        cnt = pcnt;
    }
    if (!mine) return;
    if (p.store_nodes) part_store<S>(p.nodes + off * NN, Q, team, L);
    part_store_root<S>(p, Q, team, L);
}

}  // namespace
}  // namespace pm
