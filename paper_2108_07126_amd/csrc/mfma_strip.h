// Strip teams: the FP64 MFMA engine of dimensions 33..64 (D = 64; the bounds of
// engine_bounds.hip take D = 32 too).
//
// A team of NT = D/16 waves carries a chain; wave c owns the D x 16 column
// strip [16 c, 16 c + 16) of every D x D complex matrix, NT tiles of 16 x 16 in
// the accumulator layout of v_mfma_f64_16x16x4f64 (lane 16 g + j holds rows
// g + 4 r of column j of each tile).  Two properties of that layout shape the
// engine:
//   - register r of tile k of the right factor is the B operand of a k-slice
//     as it stands, so a right factor is never staged;
//   - the A operand of S^H X needs conj(S[k][i]) for the lane's k and i = its
//     column index, which is what lane, tile and register of the same number
//     hold in the wave that owns column tile i / 16.  A left factor is staged
//     by every wave writing its registers as they are, and read back at the
//     same lane: 16-byte accesses at consecutive lanes, no padding, no bank
//     conflicts, no transposition.
// The engine therefore computes S^H X only.  That is S X for the Hermitian
// factors of the series, and for the chain it carries E = exp(i G) - I, whose
// adjoint is exp(-i G) - I: Q <- Q + E^H Q.
//
// The series is the truncated Taylor polynomial of exp(i G) in blocks of three
// powers (Paterson-Stockmeyer): Y = G G and Z = G Y, both from one staging of
// G, then a Horner step X <- B_i - i Z X per block, all from one staging of Z.
// Degree 3 (H + 1) costs 2 + H products and two stagings; with the chain's
// there are three stagings, and with two slots three barriers, per slice,
// whatever the degree.
//
// KS: the k-slices (of four rows) that the embedded dimension reaches,
// du <= 4 KS; rows and columns past them are zero in every product.
#pragma once

#include "mfma_tiles.h"

namespace pm {
namespace {

template <int NT>
struct Strip {
    Tile<double> t[NT];
};

// Per-wave coordinates: c the wave's column tile.
struct SLane {
    int lane, g, j, c;
};

template <int NT>
constexpr size_t strip_slot_bytes() {
    return (size_t)256 * NT * NT * 16;
}

// Apply f(tile, register) to every entry a lane holds.
template <int NT, class F>
__device__ __forceinline__ void strip_each(F f) {
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) f(k, r);
}

// The row of register r of tile k.
__device__ __forceinline__ int strip_row(const SLane& L, int k, int r) { return 16 * k + L.g + 4 * r; }

__device__ __forceinline__ bool strip_diag(const SLane& L, int k, int r) { return k == L.c && L.g + 4 * r == L.j; }

template <int NT>
__device__ __forceinline__ Strip<NT> strip_diagonal(const SLane& L, double v) {
    Strip<NT> s;
    strip_each<NT>([&](int k, int r) {
        s.t[k].re[r] = strip_diag(L, k, r) ? v : 0.0;
        s.t[k].im[r] = 0.0;
    });
    return s;
}

template <int NT>
__device__ __forceinline__ void strip_add(Strip<NT>& y, const Strip<NT>& x) {
    strip_each<NT>([&](int k, int r) {
        y.t[k].re[r] += x.t[k].re[r];
        y.t[k].im[r] += x.t[k].im[r];
    });
}

typedef double d2_t __attribute__((ext_vector_type(2)));

// Stage the wave's strip of a left factor (its registers as they are).
template <int NT>
__device__ __forceinline__ void strip_stage(char* slot, const Strip<NT>& S, const SLane& L) {
    d2_t* s = reinterpret_cast<d2_t*>(slot) + L.c * NT * 256 + L.lane;
    strip_each<NT>([&](int k, int r) { s[(k * 4 + r) * 64] = d2_t{S.t[k].re[r], S.t[k].im[r]}; });
}

// Position (in entries) of element (row, col) of a staged matrix.
template <int NT>
__device__ __forceinline__ int strip_at(int row, int col) {
    const int r16 = row & 15;
    return (((col >> 4) * NT + (row >> 4)) * 4 + (r16 >> 2)) * 64 + 16 * (r16 & 3) + (col & 15);
}

// Stage S^H: the products then compute S X.
template <int NT>
__device__ __forceinline__ void strip_stage_adj(char* slot, const Strip<NT>& S, const SLane& L) {
    d2_t* s = reinterpret_cast<d2_t*>(slot);
    strip_each<NT>([&](int k, int r) {
        s[strip_at<NT>(16 * L.c + L.j, strip_row(L, k, r))] = d2_t{S.t[k].re[r], -S.t[k].im[r]};
    });
}

struct NoStep {
    __device__ __forceinline__ void operator()(int) const {}
};

// S^H X for the staged S, as three real products chained through the
// accumulator: k = (Sr - Si) Xr, Re = k + Si (Xr + Xi), Im = k + Sr (Xi - Xr).
// Re and Im start from k as their MFMAs' C operand, so no sums follow the
// matrix instructions, and a row tile needs one vector operation per three
// MFMAs.  That matters: no vector instruction overlaps an FP64 MFMA of the same
// SIMD, and a SIMD with a single wave issues one in about 7 cycles.
// The next row tile's fragments are read as this one's are used up.
// step(f) is called RT * RT times among the products (work to overlap, for
// instance the next slice's basis loads).
template <int NT, int KS, class F = NoStep>
__device__ __forceinline__ Strip<NT> strip_mul(const char* slot, const Strip<NT>& X, const SLane& L,
                                               F step = F()) {
    constexpr int RT = (KS + 3) / 4;        // row tiles reached
    Strip<NT> out;
    strip_each<NT>([&](int k, int r) { out.t[k].re[r] = out.t[k].im[r] = 0.0; });
    if (L.c >= RT) return out;
    const d2_t* s = reinterpret_cast<const d2_t*>(slot) + L.lane;
    double xp[KS], xm[KS];
    d2_t a[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) a[q] = s[q * 64];
#pragma unroll
    for (int q = 0; q < KS; ++q) {
        const double xr = X.t[q >> 2].re[q & 3], xi = X.t[q >> 2].im[q & 3];
        xp[q] = xr + xi;
        xm[q] = xi - xr;
    }
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        d4_t kk = {0, 0, 0, 0};
#pragma unroll
        for (int q0 = 0; q0 < KS; q0 += 4) {
            // (a difference right before the MFMA that reads it would cost
            // wait states each time)
            double d[4];
#pragma unroll
            for (int q = q0; q < q0 + 4 && q < KS; ++q) d[q - q0] = a[q].x - a[q].y;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = q0; q < q0 + 4 && q < KS; ++q) kk = mfma16(d[q - q0], X.t[q >> 2].re[q & 3], kk);
            __builtin_amdgcn_sched_barrier(0);
        }
        d4_t re = kk, im = kk;
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            if ((q & 3) == 0) {
                __builtin_amdgcn_sched_barrier(0);
                step(i * RT + (q >> 2));
                __builtin_amdgcn_sched_barrier(0);
            }
            re = mfma16(a[q].y, xp[q], re);
            im = mfma16(a[q].x, xm[q], im);
            if (i + 1 < RT) a[q] = s[((i + 1) * NT * 4 + q) * 64];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            out.t[i].re[r] = re[r];
            out.t[i].im[r] = im[r];
        }
    }
    return out;
}

// Two LDS slots used in turn: a stage writes the slot that no wave reads any
// more (its last reads came before the barrier of the stage in between), so
// one barrier per stage suffices.
struct Slots {
    char* s[2];
    int cur;
    __device__ __forceinline__ char* next() {
        cur ^= 1;
        return cur ? s[0] : s[1];
    }
};

template <int NT>
__device__ __forceinline__ const char* strip_put(Slots& b, const Strip<NT>& S, const SLane& L) {
    char* s = b.next();
    strip_stage<NT>(s, S, L);
    __syncthreads();
    return s;
}

template <int NT>
__device__ __forceinline__ const char* strip_put_adj(Slots& b, const Strip<NT>& S, const SLane& L) {
    char* s = b.next();
    strip_stage_adj<NT>(s, S, L);
    __syncthreads();
    return s;
}

// exp(i G) - I for the (pre-scaled) Hermitian G by evaluation scheme q
// (scheme_degree(q); coefficients p.tc[k] = 1/k!, zero past the degree cap):
//   q = 0  i G;   q = 1  i G - Y/2;   q = 2  i G - Y (1/2 + i G/6 - Y/24);
//   q >= 3 blocks B_i = c_{3i} + c_{3i+1} i G - c_{3i+2} Y over powers of
//          (i G)^3 = -i Z.
template <int NT, int KS>
__device__ __forceinline__ Strip<NT> strip_expm1(const PropParams& p, const Strip<NT>& G, int q, const SLane& L,
                                                 Slots& sl) {
    Strip<NT> E;
    if (q == 0) {
        strip_each<NT>([&](int k, int r) {
            E.t[k].re[r] = -G.t[k].im[r];
            E.t[k].im[r] = G.t[k].re[r];
        });
        return E;
    }
    // c0 I + c1 i G - c2 Y into E
    auto block = [&](const Strip<NT>& Y, double c0, double c1, double c2) {
        strip_each<NT>([&](int k, int r) {
            E.t[k].re[r] = fma(-c1, G.t[k].im[r], fma(-c2, Y.t[k].re[r], strip_diag(L, k, r) ? c0 : 0.0));
            E.t[k].im[r] = fma(c1, G.t[k].re[r], -c2 * Y.t[k].im[r]);
        });
    };
    const char* s = strip_put<NT>(sl, G, L);
    const Strip<NT> Y = strip_mul<NT, KS>(s, G, L);
    if (q <= 2) {
        if (q == 1) {
            block(Y, 0.0, 1.0, p.tc[2]);
            return E;
        }
        s = strip_put<NT>(sl, Y, L);
        block(Y, p.tc[2], p.tc[3], p.tc[4]);
        E = strip_mul<NT, KS>(s, E, L);
        strip_each<NT>([&](int k, int r) {
            E.t[k].re[r] = -G.t[k].im[r] - E.t[k].re[r];
            E.t[k].im[r] = G.t[k].re[r] - E.t[k].im[r];
        });
        return E;
    }
    int i = q - 2;   // the leading block
    {
        const Strip<NT> Z = strip_mul<NT, KS>(s, Y, L);
        s = strip_put<NT>(sl, Z, L);
        block(Y, p.tc[3 * i], p.tc[3 * i + 1], p.tc[3 * i + 2]);
        const double c3 = p.tc[3 * i + 3];
        strip_each<NT>([&](int k, int r) {
            E.t[k].re[r] = fma(c3, Z.t[k].im[r], E.t[k].re[r]);
            E.t[k].im[r] = fma(-c3, Z.t[k].re[r], E.t[k].im[r]);
        });
    }
    while (--i > 0) {
        const Strip<NT> W = strip_mul<NT, KS>(s, E, L);
        block(Y, p.tc[3 * i], p.tc[3 * i + 1], p.tc[3 * i + 2]);
        strip_each<NT>([&](int k, int r) {
            E.t[k].re[r] += W.t[k].im[r];
            E.t[k].im[r] -= W.t[k].re[r];
        });
    }
    // the last block: c0 left out, c1 = 1
    const Strip<NT> W = strip_mul<NT, KS>(s, E, L);
    const double c2 = p.tc[2];
    strip_each<NT>([&](int k, int r) {
        E.t[k].re[r] = fma(-c2, Y.t[k].re[r], W.t[k].im[r]) - G.t[k].im[r];
        E.t[k].im[r] = fma(-c2, Y.t[k].im[r], G.t[k].re[r]) - W.t[k].re[r];
    });
    return E;
}

// exp(i G) - I by the degree-m Chebyshev series on the interval [-theta, theta],
// split into its even and odd halves: C + i P with C = sum e_i T_i(Y) and P = X sum b_i T_i(Y),
// X = G / theta, Y = 2 X^2 - I; `ec` the degree's row of even and odd
// coefficients.
template <int NT, int KS>
__device__ __forceinline__ Strip<NT> strip_cheb(const Strip<NT>& G, int m, double theta, const double* ec,
                                                const SLane& L, Slots& sl) {
    const double inv = 1.0 / theta;
    const double* eb = ec + kChebHalf;
    const int qc = m / 2, qs = (m - 1) / 2;
    Strip<NT> X, C = strip_diagonal<NT>(L, ec[0]), Sp = strip_diagonal<NT>(L, eb[0]);
    strip_each<NT>([&](int k, int r) {
        X.t[k].re[r] = G.t[k].re[r] * inv;
        X.t[k].im[r] = G.t[k].im[r] * inv;
    });
    auto add = [&](Strip<NT>& A, double c, const Strip<NT>& B) {
#pragma unroll
        for (int k = 0; k < NT; ++k) axpy(A.t[k], c, B.t[k]);
    };
    if (qc >= 1) {
        const char* s = strip_put<NT>(sl, X, L);
        Strip<NT> Tc = strip_mul<NT, KS>(s, X, L), Tm = strip_diagonal<NT>(L, 1.0);
        strip_each<NT>([&](int k, int r) {
            Tc.t[k].re[r] = fma(2.0, Tc.t[k].re[r], -Tm.t[k].re[r]);
            Tc.t[k].im[r] *= 2.0;
        });
        add(C, ec[1], Tc);
        if (qs >= 1) add(Sp, eb[1], Tc);
        if (qc >= 2) s = strip_put<NT>(sl, Tc, L);
        // T_i over T_{i-2}, in turns (no copies, no third strip)
        auto next = [&](int i, const Strip<NT>& T1, Strip<NT>& Tn) {
            const Strip<NT> Z = strip_mul<NT, KS>(s, T1, L);
            strip_each<NT>([&](int k, int r) {
                Tn.t[k].re[r] = fma(2.0, Z.t[k].re[r], -Tn.t[k].re[r]);
                Tn.t[k].im[r] = fma(2.0, Z.t[k].im[r], -Tn.t[k].im[r]);
            });
            add(C, ec[i], Tn);
            if (i <= qs) add(Sp, eb[i], Tn);
        };
        for (int i = 2; i <= qc; i += 2) {
            next(i, Tc, Tm);
            if (i == qc) break;
            next(i + 1, Tm, Tc);
        }
    }
    Strip<NT> P;
    if (qs >= 1) {
        P = strip_mul<NT, KS>(strip_put<NT>(sl, X, L), Sp, L);
    } else {
        strip_each<NT>([&](int k, int r) {
            P.t[k].re[r] = eb[0] * X.t[k].re[r];
            P.t[k].im[r] = eb[0] * X.t[k].im[r];
        });
    }
    strip_each<NT>([&](int k, int r) {
        C.t[k].re[r] = (C.t[k].re[r] - (strip_diag(L, k, r) ? 1.0 : 0.0)) - P.t[k].im[r];
        C.t[k].im[r] += P.t[k].re[r];
    });
    return C;
}

// The commutator [X, Y] = X Y - (X Y)^H of Hermitian X, Y: the adjoint is
// read back transposed from the product's staged copy.
template <int NT, int KS>
__device__ __forceinline__ Strip<NT> strip_commutator(const Strip<NT>& X, const Strip<NT>& Y, const SLane& L,
                                                      Slots& sl) {
    Strip<NT> Z = strip_mul<NT, KS>(strip_put<NT>(sl, X, L), Y, L);
    const d2_t* s = reinterpret_cast<const d2_t*>(strip_put<NT>(sl, Z, L));
    strip_each<NT>([&](int k, int r) {
        const d2_t a = s[strip_at<NT>(16 * L.c + L.j, strip_row(L, k, r))];
        Z.t[k].re[r] -= a.x;
        Z.t[k].im[r] += a.y;
    });
    return Z;
}

// E <- (I + E)^2 - I = 2 E + E E, s times.
template <int NT, int KS>
__device__ __forceinline__ void strip_square(Strip<NT>& E, int s, const SLane& L, Slots& sl) {
    for (int q = 0; q < s; ++q) {
        const Strip<NT> P = strip_mul<NT, KS>(strip_put_adj<NT>(sl, E, L), E, L);
        strip_each<NT>([&](int k, int r) {
            E.t[k].re[r] = fma(2.0, E.t[k].re[r], P.t[k].re[r]);
            E.t[k].im[r] = fma(2.0, E.t[k].im[r], P.t[k].im[r]);
        });
    }
}

// ||G||_1 (bound) of the Hermitian G, the same value in every wave.  red: NT
// floats of LDS.
template <int NT>
__device__ __forceinline__ double strip_norm1(const Strip<NT>& G, const SLane& L, float* red) {
    float cs = 0.0f;
    strip_each<NT>([&](int k, int r) { cs += abs_bound_f(G.t[k].re[r], G.t[k].im[r]); });
    // the column's four lane groups, then the strip's largest column
    cs += __shfl_xor(cs, 16);
    cs += __shfl_xor(cs, 32);
#pragma unroll
    for (int x = 1; x < 16; x <<= 1) cs = fmaxf(cs, __shfl_xor(cs, x));
    __syncthreads();
    if (L.lane == 0) red[L.c] = cs;
    __syncthreads();
    float m = red[0];
#pragma unroll
    for (int k = 1; k < NT; ++k) m = fmaxf(m, red[k]);
    return (double)m * (1.0 + 0x1p-16) + 0x1p-60;
}

// Node (chain or tree product) in memory: [D][D] complex128, row-major.
template <int NT>
__device__ __forceinline__ void strip_node_store(double* node, const Strip<NT>& Q, const SLane& L) {
    d2_t* o = reinterpret_cast<d2_t*>(node);
    strip_each<NT>([&](int k, int r) {
        o[strip_row(L, k, r) * (16 * NT) + 16 * L.c + L.j] = d2_t{Q.t[k].re[r], Q.t[k].im[r]};
    });
}

template <int NT>
__device__ __forceinline__ Strip<NT> strip_node_load(const double* node, const SLane& L) {
    const d2_t* o = reinterpret_cast<const d2_t*>(node);
    Strip<NT> Q;
    strip_each<NT>([&](int k, int r) {
        const d2_t v = o[strip_row(L, k, r) * (16 * NT) + 16 * L.c + L.j];
        Q.t[k].re[r] = v.x;
        Q.t[k].im[r] = v.y;
    });
    return Q;
}

// The adjoint of a node: the left factor X of X P is staged as X^H.
template <int NT>
__device__ __forceinline__ Strip<NT> strip_node_load_adj(const double* node, const SLane& L) {
    const d2_t* o = reinterpret_cast<const d2_t*>(node);
    Strip<NT> Q;
    strip_each<NT>([&](int k, int r) {
        const d2_t v = o[(16 * L.c + L.j) * (16 * NT) + strip_row(L, k, r)];
        Q.t[k].re[r] = v.x;
        Q.t[k].im[r] = -v.y;
    });
    return Q;
}

// Take the identity from a staged node (the wave that staged its diagonal entries
// does, before the barrier): the tree joins nodes as X + (A - I) X, which rounds
// relative to ||A - I|| (mx_join in mfma_wave.h).
template <int NT>
__device__ __forceinline__ void strip_staged_less_one(char* slot, const SLane& L) {
    double* s = reinterpret_cast<double*>(slot);
    if (L.lane < 16) s[2 * strip_at<NT>(16 * L.c + L.lane, 16 * L.c + L.lane)] -= 1.0;
}

template <int NT, int KS, bool JOIN>
__device__ __forceinline__ Strip<NT> strip_node_mul(const char* s, const Strip<NT>& X, const SLane& L) {
    Strip<NT> y = strip_mul<NT, KS>(s, X, L);
    if constexpr (JOIN) strip_add<NT>(y, X);
    return y;
}

// Root product into U_out.
template <int NT>
__device__ __forceinline__ void strip_store_root(const PropParams& p, const Strip<NT>& Q, const SLane& L) {
    const int col = 16 * L.c + L.j;
    if (col >= p.du) return;
    strip_each<NT>([&](int k, int r) {
        const int row = strip_row(L, k, r);
        if (row < p.du) {
            p.U_out[(row * p.du + col) * 2 + 0] = Q.t[k].re[r];
            p.U_out[(row * p.du + col) * 2 + 1] = Q.t[k].im[r];
        }
    });
}

// The ticketed product tree of strip teams: a team stores its node, releases it
// and takes its group's ticket; the last arrival multiplies the group's nodes and
// goes on.  A 64 x 64 product takes a CU 5 us and a level's stores, fences and
// loads about as much, so the groups are pairs (own node in registers): for 512
// chains 9 products one after another instead of the 21 of fan-in 8 (2048
// slices of 64 levels in FP32 550 -> 437 us, in BF16 split 350 -> 292 us).  With p.store_nodes the groups are the
// kFanIn nodes that the checkpoints are assembled from, multiplied the earliest
// first, each left factor's adjoint read straight from memory.  Waves past the
// strips (active false) only keep the barriers.
// JOIN: nodes are joined as X + (A - I) X.  (The reduced precisions' chains round a
// million times more, and their two waves per SIMD have no registers for X beside
// the product: 65536 slices of 64 levels in BF16 split 2854 us, with JOIN 2961.)
template <int NT, int KS, bool JOIN>
__device__ void strip_tree(const PropParams& p, int64_t leaf, Strip<NT> Q, const SLane& L, Slots& sl, int* tick,
                           bool active = true) {
    constexpr int64_t NN = (int64_t)256 * NT * NT * 2;
    const int shift = p.store_nodes ? kFanInLog2 : 1;
    const int64_t fan = (int64_t)1 << shift;
    int64_t idx = leaf, cnt = p.n_leaves, off = 0;
    while (cnt > 1) {
        const int64_t pcnt = (cnt + fan - 1) >> shift, poff = off + cnt, grp = idx >> shift;
        const int64_t first = grp << shift;
        const int64_t members = min(cnt, first + fan) - first;
        if (active && (members > 1 || p.store_nodes)) strip_node_store<NT>(p.nodes + (off + idx) * NN, Q, L);
        if (members > 1) {
            __syncthreads();   // every wave's part of the node is stored
            if (active && L.c == 0 && L.lane == 0) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                const unsigned v = atomicAdd(&p.counters[poff + grp], 1u);
                if (v == (unsigned)(members - 1)) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                    atomicExch(&p.counters[poff + grp], 0u);
                }
                *tick = (int)v;
            }
            __syncthreads();
            const int t = wave_uniform(*tick);
            __syncthreads();
            if (t != (int)(members - 1)) return;
            if (members == 2) {
                char* s = sl.next();
                if (active) {
                    if (idx == first) {
                        strip_stage<NT>(s, strip_node_load_adj<NT>(p.nodes + (off + first + 1) * NN, L), L);
                    } else {
                        strip_stage_adj<NT>(s, Q, L);
                        Q = strip_node_load<NT>(p.nodes + (off + first) * NN, L);
                    }
                    if constexpr (JOIN) strip_staged_less_one<NT>(s, L);
                }
                __syncthreads();
                if (active) Q = strip_node_mul<NT, KS, JOIN>(s, Q, L);
            } else {
                if (active) Q = strip_node_load<NT>(p.nodes + (off + first) * NN, L);
                for (int64_t k = first + 1; k < first + members; ++k) {
                    char* s = sl.next();
                    if (active) {
                        strip_stage<NT>(s, strip_node_load_adj<NT>(p.nodes + (off + k) * NN, L), L);
                        if constexpr (JOIN) strip_staged_less_one<NT>(s, L);
                    }
                    __syncthreads();
                    if (active) Q = strip_node_mul<NT, KS, JOIN>(s, Q, L);
                }
            }
        }
        idx = grp;
        off = poff;
        cnt = pcnt;
    }
    if (!active) return;
    if (p.store_nodes) strip_node_store<NT>(p.nodes + off * NN, Q, L);
    strip_store_root<NT>(p, Q, L);
}

}  // namespace
}  // namespace pm
