// Panel teams: the reduced-precision MFMA engine of dimensions 33..64.
//
// A chain runs on a block of eight waves, one block per CU, as two teams of four:
// of every two slices each team exponentiates one, then all eight waves multiply
// both into the chain product.  The exponentials of different slices are
// independent, only the chain product is serial, so a CU works on two slices
// while the chains (and with them every rounding of the FP32 arithmetic) stay
// as long as one chain per CU makes them.
//
// Wave w of a team owns the 16 x 64 row panel [16 w, 16 w + 16) of the slice's
// matrices, tile k transposed in registers: lane 16 g + j holds row 16 w + j,
// columns 16 k + 4 g + r (r = 0..3).  The accumulator of an MFMA whose *first*
// operand is the right factor's columns and whose second is the panel's rows
// has exactly that layout, and then
//   - the left factor of a product is the wave's own panel: a 4 x 4 exchange
//     between lane groups (v_permlane32/16_swap) turns its registers into
//     operand fragments, no LDS and no barrier;
//   - the right factor is staged as rows, four consecutive entries per lane in
//     one write (BF16 split: hi and lo planes split once at staging).
// The powers Y^k = Y^{k-1} Y need no staging past Y, so a slice has four (G, Y,
// the sine series, E) whatever its degree.  The chain product Q is held by
// columns: wave (c, half) owns rows [32 half, 32 half + 32) of the strip of
// columns [16 c, 16 c + 16), in FP64; E is the staged left factor and Q's rounded
// halves are exchanged as operand fragments.  Six barriers per two slices.
//
// Bounds: in BF16 split vector issue (splits, scaling, the expansion) and LDS reads
// beside the matrix cores, in FP32 the matrix cores, which share the vector
// units.  Against one tile per wave on 16 waves, both factors of every product
// staged and read back, 12 barriers per slice: 65536 slices of 64 levels in BF16
// split 4850 -> 3000 us, FP32 8580 -> 7400 us, FP32-3M 7510 -> 6570 us; 16384
// fourth-order slices with four controls (15 basis matrices) in BF16 split 3390
// -> 1310 us.  The products, their operand order and the order of every sum
// are those of mfma_tiles.h, so results agree to the last FP32 bit.
//
// Two things cost more than they look.  Registers: the 256 of a wave are just
// enough, and a spill waits behind the basis loads in flight (memory operations
// return in order), so lane coordinates are re-formed (fresh) instead of letting
// addresses be hoisted, and each degree class has its own straight-line path.
// HBM latency: samples are turned into weights 32 slices at a time (panel_run).
#pragma once

#include "mfma_strip.h"

namespace pm {
namespace {

constexpr int kPanelD = 64;
constexpr int kPanelSlot = 2 * kPanelD * kPanelD * 4;       // bytes: two FP32 planes or four BF16 planes
constexpr int kPanelRootLd = kPanelD + 1;
static_assert(2 * kPanelD * kPanelD * 8 <= 2 * kPanelSlot, "a team's FP64 matrix takes two slots");
static_assert(kPanelD * kPanelRootLd * 16 <= 4 * kPanelSlot, "the chain product");
static_assert(2 * strip_slot_bytes<4>() <= 4 * kPanelSlot, "the tree's slots");
constexpr int kPanelAhead = 32;   // slices whose weights are in LDS at a time
constexpr size_t kPanelLds = 4 * kPanelSlot + (2 * 2 * 2 * kPanelD + kPanelAhead * kMaxBasis) * sizeof(double) + 16;
static_assert(kPanelLds <= 160 * 1024, "the CU's LDS");

// Per-wave coordinates: team, panel w (rows of the exponentials), column strip
// c and half of the chain product.
struct PLane {
    int lane, g, j, team, w;
};

// The same coordinates, opaque to the optimiser: what is computed from them (LDS
// addresses, diagonal masks) is formed again where it is used instead of being
// kept for the whole chain, for which there are no registers.
__device__ __forceinline__ PLane fresh(const PLane& L) {
    PLane F = L;
    asm volatile("" : "+v"(F.lane));
    F.g = F.lane >> 4;
    F.j = F.lane & 15;
    return F;
}

struct Panel {
    Tile<float> t[4];
};

template <class F>
__device__ __forceinline__ void panel_each(F f) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) f(k, r);
}

__device__ __forceinline__ bool panel_diag(const PLane& L, int k, int r) { return k == L.w && 4 * L.g + r == L.j; }

// Exchange between the lane groups g (rows of 16 lanes): a and b become
// {a0, a2, b0, b2} and {a1, a3, b1, b3}, x_g the value of group g.
__device__ __forceinline__ void swap_pairs(unsigned& a, unsigned& b) {
    const auto u = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    const auto v = __builtin_amdgcn_permlane16_swap(u[0], u[1], false, false);
    a = v[0];
    b = v[1];
}

// Transpose of registers and lane groups: x[q] of group g becomes x[g] of group q.
__device__ __forceinline__ void swap_transpose(float (&x)[4]) {
    unsigned u[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] = __float_as_uint(x[q]);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const auto s = __builtin_amdgcn_permlane32_swap(u[q], u[q + 2], false, false);
        u[q] = s[0];
        u[q + 2] = s[1];
    }
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
        const auto s = __builtin_amdgcn_permlane16_swap(u[q], u[q + 1], false, false);
        u[q] = s[0];
        u[q + 1] = s[1];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = __uint_as_float(u[q]);
}

// Operand fragments over 32 values of k of the line (row or column) that a
// lane's j stands for.  BF16 split: eight consecutive k = 32 b + 8 g + q, real hi,
// lo, imaginary hi, lo; FP32: k = 4 kb + g, eight kb, real then imaginary.
template <int PMODE>
struct Frag;
template <>
struct Frag<2> {
    bf8_t x[4];
};
template <>
struct Frag<0> {
    float re[8], im[8];
};
template <>
struct Frag<1> : Frag<0> {};

struct PanelU2 {
    unsigned x, y;
};

// The split of an FP64 tile: lo takes what hi leaves of the FP32 rounding, and hi
// is rounded from the FP64 value itself.  That differs from rounding the FP32
// value only where it lies halfway between two BF16 values and the FP64 value
// does not: hi is then rounded from the FP32 neighbour towards the FP64 value
// (a rare path).
struct SplitTile {
    Split4 re, im;
};

__device__ __forceinline__ SplitTile split_tile(const Tile<double>& x) {
    float f[8], t[8];
    unsigned tie = ~0u;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        f[q] = (float)(q < 4 ? x.re[q] : x.im[q - 4]);
        asm("" : "+v"(f[q]));
        t[q] = f[q];
        tie = min(tie, (__float_as_uint(f[q]) << 16) ^ 0x80000000u);
    }
    if (__ballot(tie == 0) != 0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double d = q < 4 ? x.re[q] : x.im[q - 4];
            const unsigned u = __float_as_uint(f[q]);
            const bool up = fabs(d) > fabs((double)f[q]);
            t[q] = __uint_as_float((u & 0xffffu) == 0x8000u && (double)f[q] != d ? (up ? u + 1u : u - 1u) : u);
        }
    }
    SplitTile s;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const __bf16 h = (__bf16)t[q], g = (__bf16)t[4 + q];
        s.re.hi[q] = h;
        s.re.lo[q] = (__bf16)(f[q] - (float)h);
        s.im.hi[q] = g;
        s.im.lo[q] = (__bf16)(f[4 + q] - (float)g);
    }
    return s;
}

__device__ __forceinline__ SplitTile split_tile(const Tile<float>& x) { return {split4(x.re), split4(x.im)}; }

// Fragments of the lane's own line from two tiles (entries 16 t + 4 g + r).
template <int PMODE, typename T>
__device__ __forceinline__ Frag<PMODE> panel_frag(const Tile<T>& t0, const Tile<T>& t1) {
    Frag<PMODE> f;
    if constexpr (PMODE == 2) {
        const SplitTile s0 = split_tile(t0), s1 = split_tile(t1);
        const Split4 a[2] = {s0.re, s0.im}, b[2] = {s1.re, s1.im};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            PanelU2 u = __builtin_bit_cast(PanelU2, c & 1 ? a[c >> 1].lo : a[c >> 1].hi);
            PanelU2 v = __builtin_bit_cast(PanelU2, c & 1 ? b[c >> 1].lo : b[c >> 1].hi);
            swap_pairs(u.x, v.x);
            swap_pairs(u.y, v.y);
            f.x[c] = cat8(__builtin_bit_cast(bf4_t, u), __builtin_bit_cast(bf4_t, v));
        }
    } else {
        float x[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            x[0][r] = (float)t0.re[r];
            x[1][r] = (float)t1.re[r];
            x[2][r] = (float)t0.im[r];
            x[3][r] = (float)t1.im[r];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) swap_transpose(x[q]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f.re[r] = x[0][r];
            f.re[4 + r] = x[1][r];
            f.im[r] = x[2][r];
            f.im[4 + r] = x[3][r];
        }
    }
    return f;
}

// Places in a slot, whose planes have no padding: an entry's position within its
// row is permuted by the row number so that rows read at one column and columns
// read at one row, eight or four lanes of 16 bytes at a time in whatever order
// the LDS takes them, fall into different banks (padding by 16 bytes left every
// second read of BF16 rows waiting for another).
// BF16: entry 8 chunk of a row, in bytes from the plane.
__device__ __forceinline__ int bf16_at(int row, int chunk) { return row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4); }
constexpr int kBfPlane = kPanelD * kPanelD * 2;

// FP32, in entries.
__device__ __forceinline__ int f32_at(int row, int col) {
    return row * kPanelD + (col ^ (((row & 3) << 4) | (((row >> 2) & 3) << 2)));
}
constexpr int kF32Plane = kPanelD * kPanelD;

// FP64 (squarings), in entries.
__device__ __forceinline__ int f64_at(int row, int col) { return row * kPanelD + (col ^ ((row & 15) << 2)); }

// The same fragments read from row 16 x + j of a slot.
template <int PMODE>
__device__ __forceinline__ Frag<PMODE> panel_frag_row(const char* slot, int x, int b, const PLane& L) {
    Frag<PMODE> f;
    if constexpr (PMODE == 2) {
        const char* p = slot + x * 16 * 128 + bf16_at(L.j, 4 * b + L.g);
#pragma unroll
        for (int c = 0; c < 4; ++c) f.x[c] = *reinterpret_cast<const bf8_t*>(p + c * kBfPlane);
    } else {
        const float* p = reinterpret_cast<const float*>(slot) + x * 16 * kPanelD;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int at = f32_at(L.j, 32 * b + 4 * q + L.g);
            f.re[q] = p[at];
            f.im[q] = p[kF32Plane + at];
        }
    }
    return f;
}

// Fragments of column 16 x + j of the matrix staged in a slot.  BF16 split: of a
// Hermitian matrix, whose column is the conjugate of its row (the sign of the
// imaginary part is the caller's).
template <int PMODE>
__device__ __forceinline__ Frag<PMODE> panel_frag_col(const char* slot, int x, int b, const PLane& L) {
    if constexpr (PMODE == 2) {
        return panel_frag_row<PMODE>(slot, x, b, L);
    } else {
        Frag<PMODE> f;
        const float* p = reinterpret_cast<const float*>(slot) + 32 * b * kPanelD;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            // row 32 b + 4 q + g
            const int at = 16 * (q >> 2) * kPanelD + f32_at(4 * (q & 3) + L.g, 16 * x + L.j);
            f.re[q] = p[at];
            f.im[q] = p[kF32Plane + at];
        }
        return f;
    }
}

// Stage tile k of the wave's panel as rows.
template <int PMODE>
__device__ __forceinline__ void panel_stage_tile(char* slot, const Tile<float>& X, int k, const PLane& L) {
    if constexpr (PMODE == 2) {
        char* p = slot + L.w * 16 * 128 + bf16_at(L.j, 2 * k + (L.g >> 1)) + 8 * (L.g & 1);
        const Split4 sr = split4(X.re), si = split4(X.im);
        *reinterpret_cast<bf4_t*>(p) = sr.hi;
        *reinterpret_cast<bf4_t*>(p + kBfPlane) = sr.lo;
        *reinterpret_cast<bf4_t*>(p + 2 * kBfPlane) = si.hi;
        *reinterpret_cast<bf4_t*>(p + 3 * kBfPlane) = si.lo;
    } else {
        float* p = reinterpret_cast<float*>(slot) + L.w * 16 * kPanelD + f32_at(L.j, 16 * k + 4 * L.g);
        *reinterpret_cast<f4_t*>(p) = f4_t{X.re[0], X.re[1], X.re[2], X.re[3]};
        *reinterpret_cast<f4_t*>(p + kF32Plane) = f4_t{X.im[0], X.im[1], X.im[2], X.im[3]};
    }
}

template <int PMODE>
__device__ __forceinline__ void panel_stage(char* slot, const Panel& X, const PLane& L) {
#pragma unroll
    for (int k = 0; k < 4; ++k) panel_stage_tile<PMODE>(slot, X.t[k], k, L);
}

// The real sums of one output tile of a complex product.
template <int PMODE>
struct PanelAcc {
    f4_t a[PMODE == 2 ? 4 : (PMODE == 1 ? 3 : 2)];
};

// Add 32 values of k (b: which), `l` the left factor's fragments (rows) and `r`
// the right one's (columns).  SWAP: the right factor is the MFMA's first
// operand (the tile comes out transposed).  The operation order is that of
// slot_mul4 (PMODE 0), slot_mul_3m (1) and slot_mul_bf16x (2).
template <int PMODE, int RT, bool SWAP>
__device__ __forceinline__ void panel_step(PanelAcc<PMODE>& c, const Frag<PMODE>& l, const Frag<PMODE>& r, int b) {
    if constexpr (PMODE == 2) {
        auto mm = [](bf8_t x, bf8_t y, f4_t z) { return SWAP ? mfma_bf16x32(y, x, z) : mfma_bf16x32(x, y, z); };
        const bf8_t arh = l.x[0], arl = l.x[1], aih = l.x[2], ail = l.x[3];
        const bf8_t brh = r.x[0], brl = r.x[1], bih = r.x[2], bil = r.x[3];
        c.a[0] = mm(arh, brh, c.a[0]);
        c.a[1] = mm(aih, bih, c.a[1]);
        c.a[2] = mm(arh, bih, c.a[2]);
        c.a[3] = mm(aih, brh, c.a[3]);
        c.a[0] = mm(arh, brl, c.a[0]);
        c.a[1] = mm(aih, bil, c.a[1]);
        c.a[2] = mm(arh, bil, c.a[2]);
        c.a[3] = mm(aih, brl, c.a[3]);
        c.a[0] = mm(arl, brh, c.a[0]);
        c.a[1] = mm(ail, bih, c.a[1]);
        c.a[2] = mm(arl, bih, c.a[2]);
        c.a[3] = mm(ail, brh, c.a[3]);
    } else {
        auto mm = [](float x, float y, f4_t z) { return SWAP ? mfma16(y, x, z) : mfma16(x, y, z); };
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (8 * b + q >= 4 * RT) break;
            const float ar = l.re[q], ai = l.im[q], br = r.re[q], bi = r.im[q];
            if constexpr (PMODE == 0) {
                c.a[0] = mm(ar, br, c.a[0]);
                c.a[1] = mm(ar, bi, c.a[1]);
                c.a[0] = mm(-ai, bi, c.a[0]);
                c.a[1] = mm(ai, br, c.a[1]);
            } else {
                c.a[0] = mm(ar, br, c.a[0]);
                c.a[1] = mm(ai, bi, c.a[1]);
                c.a[2] = mm(ar + ai, br + bi, c.a[2]);
            }
        }
    }
}

// The tile from its sums.  HERM (BF16 split): the right fragments are conjugated.
template <int PMODE, bool HERM>
__device__ __forceinline__ Tile<float> panel_tile(const PanelAcc<PMODE>& c) {
    Tile<float> out;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if constexpr (PMODE == 2) {
            out.re[q] = HERM ? c.a[0][q] + c.a[1][q] : c.a[0][q] - c.a[1][q];
            out.im[q] = HERM ? c.a[3][q] - c.a[2][q] : c.a[2][q] + c.a[3][q];
        } else if constexpr (PMODE == 1) {
            out.re[q] = c.a[0][q] - c.a[1][q];
            out.im[q] = c.a[2][q] - c.a[0][q] - c.a[1][q];
        } else {
            out.re[q] = c.a[0][q];
            out.im[q] = c.a[1][q];
        }
    }
    return out;
}

// Vector and scalar operations may cross, matrix and memory operations stay.
__device__ __forceinline__ void panel_pin() { __builtin_amdgcn_sched_barrier(0x2 | 0x4); }

// X B for the own panel's fragments and the staged B (BF16 split: Hermitian);
// each output tile goes to f(k, tile), zero past the embedded dimension.  The
// next 32 values' fragments are read behind the MFMAs of the current ones.
template <int PMODE, int RT, class F>
__device__ __forceinline__ void panel_mul(const Frag<PMODE> (&x)[2], const char* slot, const PLane& L, F f) {
    if constexpr (RT < 4) {
        Tile<float> o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o.re[r] = o.im[r] = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k >= RT || L.w >= RT) f(k, o);
        if (L.w >= RT) return;
    }
    Frag<PMODE> cur = panel_frag_col<PMODE>(slot, 0, 0, L);
#pragma unroll
    for (int k = 0; k < RT; ++k) {
        PanelAcc<PMODE> c{};
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            Frag<PMODE> nxt;
            if (2 * k + b + 1 < 2 * RT)
                nxt = panel_frag_col<PMODE>(slot, b ? k + 1 : k, b ^ 1, L);
            panel_pin();
            panel_step<PMODE, RT, true>(c, x[b], cur, b);
            panel_pin();
            cur = nxt;
        }
        f(k, panel_tile<PMODE, true>(c));
    }
}

template <int PMODE>
__device__ __forceinline__ void panel_own(Frag<PMODE> (&x)[2], const char* slot, const PLane& L) {
#pragma unroll
    for (int b = 0; b < 2; ++b) x[b] = panel_frag_row<PMODE>(slot, L.w, b, L);
}

// The exponents of a pair of slices.  Wave w of team h forms tiles 2 h and 2 h + 1 of
// row panel w for both slices, so the block reads each basis entry once per
// pair.  A tile's first four basis matrices are requested (issue) a stage before
// they are used (consume): the loads' latency passes behind the chain
// product's MFMAs.
struct PanelExpand {
    double x[4][8];
    Tile<float> G[2][2]; // [slice][tile]
    double rs[2];        // partial row sums of the entries' bounds

    // basis matrices m0 .. m0 + 3 of a tile (uniform base and lane offset apart:
    // one register for all addresses)
    static __device__ __forceinline__ void load(const PropParams& p, double (&y)[4][8], int kk, int m0, const PLane& L) {
        const unsigned off = (unsigned)L.lane * 8u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const char* bm = reinterpret_cast<const char*>(
                p.basis + mfma_basis_index(kPanelD, min(m0 + q, p.M - 1), 2 * L.team + kk, L.w, 0, 0, 0));
#pragma unroll
            for (int e = 0; e < 8; ++e) y[q][e] = *reinterpret_cast<const double*>(bm + off + e * 512);
        }
    }
    // w: the weights of the first slice, those of the second p.M further
    static __device__ __forceinline__ void add(const PropParams& p, double (&g)[2][8], const double (&y)[4][8], int m0,
                                               const double* w) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int m = m0 + q < p.M ? m0 + q : 0;
                const double wm = m0 + q < p.M ? w[t * p.M + m] : 0.0;
#pragma unroll
                for (int e = 0; e < 8; ++e) g[t][e] = fma(wm, y[q][e], g[t][e]);
            }
    }
    __device__ __forceinline__ void issue(const PropParams& p, int kk, const PLane& L) { load(p, x, kk, 0, L); }
    // FP64 sums in order of the basis, then FP32.  The basis is Hermitian to the
    // last bit: the transposed tile (w, k) is the conjugate of tile (k, w).
    __device__ __forceinline__ void consume(const PropParams& p, int kk, const double* w, const PLane& L) {
        double g[2][8] = {};
        add(p, g, x, 0, w);
        for (int m0 = 4; m0 < p.M; m0 += 4) {
            double y[4][8];
            load(p, y, kk, m0, L);
            add(p, g, y, m0, w);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                rs[t] += abs_bound(g[t][r], g[t][4 + r]);
                float re = (float)g[t][r], im = -(float)g[t][4 + r];
                // (values of their own: a BF16 rounding of G starts from them,
                // not from the FP64 sums)
                asm("" : "+v"(re), "+v"(im));
                G[t][kk].re[r] = re;
                G[t][kk].im[r] = im;
            }
    }
};

// E <- (I + E)^2 - I = 2E + E E, s times in FP64 (`rounds` the larger s of the
// two teams, whose barriers run together).
__device__ __forceinline__ void panel_square(Panel& E, int s, int rounds, char* lds, PLane L) {
    L = fresh(L);
    double* re = reinterpret_cast<double*>(lds + L.team * 2 * kPanelSlot);
    double* im = re + kPanelD * kPanelD;
    const int row = 16 * L.w + L.j;
    __syncthreads();
    panel_each([&](int k, int r) {
        re[f64_at(row, 16 * k + 4 * L.g + r)] = (double)E.t[k].re[r];
        im[f64_at(row, 16 * k + 4 * L.g + r)] = (double)E.t[k].im[r];
    });
    __syncthreads();
    for (int i = 0; i < rounds; ++i) {
        Tile<double> P[4];
        if (i < s) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                d4_t t1 = {0, 0, 0, 0}, t2 = {0, 0, 0, 0}, t3 = {0, 0, 0, 0};
#pragma unroll 4
                for (int kb = 0; kb < 16; ++kb) {
                    const int c = 4 * kb + L.g, own = f64_at(row, c), at = f64_at(c, 16 * k + L.j);
                    const double ar = re[own], ai = im[own], br = re[at], bi = im[at];
                    t1 = mfma16(br, ar, t1);
                    t2 = mfma16(bi, ai, t2);
                    t3 = mfma16(br + bi, ar + ai, t3);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int at = f64_at(row, 16 * k + L.g + 4 * r);
                    P[k].re[r] = fma(2.0, re[at], t1[r] - t2[r]);
                    P[k].im[r] = fma(2.0, im[at], t3[r] - t1[r] - t2[r]);
                }
            }
        }
        __syncthreads();
        if (i < s)
            panel_each([&](int k, int r) {
                re[f64_at(row, 16 * k + L.g + 4 * r)] = P[k].re[r];
                im[f64_at(row, 16 * k + L.g + 4 * r)] = P[k].im[r];
            });
        __syncthreads();
    }
    if (s > 0)
        panel_each([&](int k, int r) {
            E.t[k].re[r] = (float)re[f64_at(row, 16 * k + 4 * L.g + r)];
            E.t[k].im[r] = (float)im[f64_at(row, 16 * k + 4 * L.g + r)];
        });
    __syncthreads();
}

// Per-slice output I + E: a lane's four entries of a row are contiguous.
__device__ __forceinline__ void panel_store_slice(const PropParams& p, int64_t j, const Panel& E, PLane L) {
    L = fresh(L);
    const int row = 16 * L.w + L.j;
    if (row >= p.du) return;
    char* out = reinterpret_cast<char*>(p.slices_out) + j * p.du * p.du * 8;
    const unsigned off = (unsigned)(row * p.du + 4 * L.g) * 8u;
    panel_each([&](int k, int r) {
        if (16 * k + 4 * L.g + r < p.du)
            *reinterpret_cast<float2*>(out + off + (16 * k + r) * 8) =
                float2{E.t[k].re[r] + (panel_diag(L, k, r) ? 1.0f : 0.0f), E.t[k].im[r]};
    });
}

// Q <- Q + E Q for the staged E; Q's rounded halves are exchanged through `ex`
// (a fragment set per wave), one barrier.
template <int PMODE, int RT>
__device__ __forceinline__ void panel_chain(Tile<double> (&Q)[2], const char* slotE, char* ex, const PLane& L) {
    struct alignas(16) U4 {
        unsigned x[4];
    };
    struct F4 {
        U4 x[4];
    };
    static_assert(sizeof(Frag<PMODE>) == sizeof(F4), "four 16-byte pieces");
    U4* e = reinterpret_cast<U4*>(ex) + L.lane;
    {
        const F4 f = __builtin_bit_cast(F4, panel_frag<PMODE>(Q[0], Q[1]));
#pragma unroll
        for (int c = 0; c < 4; ++c) e[((L.team * 4 + L.w) * 4 + c) * 64] = f.x[c];
    }
    __syncthreads();
    if (RT == 4 || L.w < RT) {
        Frag<PMODE> q[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            F4 v;
#pragma unroll
            for (int c = 0; c < 4; ++c) v.x[c] = e[((b * 4 + L.w) * 4 + c) * 64];
            q[b] = __builtin_bit_cast(Frag<PMODE>, v);
        }
        Frag<PMODE> cur = panel_frag_row<PMODE>(slotE, 2 * L.team, 0, L);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (RT < 4 && 2 * L.team + i >= RT) break;
            PanelAcc<PMODE> c{};
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                Frag<PMODE> nxt;
                if (2 * i + b < 3)
                    nxt = panel_frag_row<PMODE>(slotE, 2 * L.team + (b ? i + 1 : i), b ^ 1, L);
                panel_pin();
                panel_step<PMODE, RT, false>(c, cur, q[b], b);
                panel_pin();
                cur = nxt;
            }
            const Tile<float> o = panel_tile<PMODE, false>(c);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                Q[i].re[r] += (double)o.re[r];
                Q[i].im[r] += (double)o.im[r];
            }
        }
    }
}

// Y = G G scaled by 4^-s from the staged G; each tile goes to f(k, tile).
template <int PMODE, int RT, class F>
__device__ __forceinline__ void panel_y(int s, const char* s0, const PLane& L, F f) {
    Frag<PMODE> x[2];
    panel_own<PMODE>(x, s0, L);
    const float sc = ldexpf(1.0f, -2 * s);
    panel_mul<PMODE, RT>(x, s0, L, [&](int k, Tile<float> o) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            o.re[r] *= sc;
            o.im[r] *= sc;
        }
        f(k, o);
    });
}

// The first terms of the cosine series (without I) and of the sine series.
__device__ __forceinline__ void panel_first(Tile<float>& C, Tile<float>& Sp, const Tile<float>& Y, int k,
                                            const PLane& L) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        C.re[r] = C.im[r] = 0.0f;
        Sp.re[r] = panel_diag(L, k, r) ? 1.0f : 0.0f;
        Sp.im[r] = 0.0f;
    }
    axpy(C, cos_coef(1), Y);
    axpy(Sp, sin_coef(1), Y);
}

// C <- C - i 2^-s G S' for the staged S' and the own panel's fragments x of G;
// each tile of the result is staged in s1.
template <int PMODE, int RT>
__device__ __forceinline__ void panel_sine(Panel& C, const Frag<PMODE> (&x)[2], int s, const char* s0, char* s1,
                                           const PLane& L) {
    const float f = ldexpf(1.0f, -s);
    panel_mul<PMODE, RT>(x, s0, L, [&](int k, const Tile<float>& o) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            C.t[k].re[r] = fmaf(f, o.im[r], C.t[k].re[r]);
            C.t[k].im[r] = fmaf(-f, o.re[r], C.t[k].im[r]);
        }
        panel_stage_tile<PMODE>(s1, C.t[k], k, L);
    });
}

// exp(-i G) - I by the Taylor polynomial of degree m >= 4 of the staged G (slot
// s0; s1 is free), scaled by 2^-s; the result is staged in s1.  Tiles are
// staged as they come out of a product, behind the next tile's MFMAs.
template <int PMODE, int RT>
__device__ __forceinline__ void panel_series(int m, int s, bool low, char* s0, char* s1, PLane L, Panel& C) {
    const int qc = m / 2, qs = (m - 1) / 2;   // highest powers of Y in the cosine and sine series
    if (low) __syncthreads();
    Panel Sp;
    panel_y<PMODE, RT>(s, s0, L, [&](int k, const Tile<float>& o) {
        panel_first(C.t[k], Sp.t[k], o, k, L);
        panel_stage_tile<PMODE>(s1, o, k, L);
    });
    L = fresh(L);
    __syncthreads();
    Frag<PMODE> x[2];
    panel_own<PMODE>(x, s1, L);
    for (int i = 2; i < qc; ++i) {
        Panel P;
        const double cc = cos_coef(i), sc = sin_coef(i);
        L = fresh(L);
        panel_mul<PMODE, RT>(x, s1, L, [&](int k, const Tile<float>& o) {
            P.t[k] = o;
            axpy(C.t[k], cc, o);
            axpy(Sp.t[k], sc, o);
        });
        x[0] = panel_frag<PMODE>(P.t[0], P.t[1]);
        x[1] = panel_frag<PMODE>(P.t[2], P.t[3]);
    }
    L = fresh(L);
    Frag<PMODE> g[2];
    panel_own<PMODE>(g, s0, L);
    {
        // (an even degree's sine series ends a term earlier)
        const double cc = cos_coef(qc), sc = qc <= qs ? sin_coef(qc) : 0.0;
        panel_mul<PMODE, RT>(x, s1, L, [&](int k, const Tile<float>& o) {
            axpy(C.t[k], cc, o);
            axpy(Sp.t[k], sc, o);
            panel_stage_tile<PMODE>(s0, Sp.t[k], k, L);
        });
    }
    __syncthreads();
    panel_sine<PMODE, RT>(C, g, s, s0, s1, L);
}

// The same for degrees 1 to 3 (mm: the larger degree of the two teams).  Degrees
// 1 and 2 take G from slot s1 (low).
template <int PMODE, int RT>
__device__ __forceinline__ void panel_short_series(int m, int s, int mm, bool low, char* s0, char* s1, PLane L,
                                                   Panel& C) {
    if (m <= 2) {
        // -i G
        const f4_t* v = reinterpret_cast<const f4_t*>(s1) + (L.w * 4 * 64 + L.lane) * 2;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const f4_t re = v[k * 128], im = v[k * 128 + 1];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                C.t[k].re[r] = ldexpf(im[r], -s);
                C.t[k].im[r] = ldexpf(-re[r], -s);
            }
        }
    }
    if (low) __syncthreads();
    Panel Y;
    if (m >= 2) panel_y<PMODE, RT>(s, s0, L, [&](int k, const Tile<float>& o) { Y.t[k] = o; });
    L = fresh(L);
    if (mm >= 4) __syncthreads();
    if (m == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            Tile<float> c;
#pragma unroll
            for (int r = 0; r < 4; ++r) c.re[r] = c.im[r] = 0.0f;
            axpy(c, cos_coef(1), Y.t[k]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                C.t[k].re[r] += c.re[r];
                C.t[k].im[r] += c.im[r];
            }
        }
    }
    if (mm == 3) __syncthreads();   // (a degree of 4 or more stages Y: that barrier comes after G's readers)
    if (m == 3) {
        Panel Sp;
#pragma unroll
        for (int k = 0; k < 4; ++k) panel_first(C.t[k], Sp.t[k], Y.t[k], k, L);
        Frag<PMODE> x[2];
        panel_own<PMODE>(x, s0, L);
        panel_stage<PMODE>(s0, Sp, L);
        __syncthreads();
        panel_sine<PMODE, RT>(C, x, s, s0, s1, L);
    } else {
        if (mm >= 3) __syncthreads();
        panel_stage<PMODE>(s1, C, L);
    }
}

// plan_expm_lanes for two slices at once, lanes 0..31 for the first and 32..63
// for the second: the own team's plan and the other's.
__device__ __forceinline__ void panel_plan(const PropParams& p, double nu0, double nu1, int lane, double lane_theta,
                                           int team, int& m, int& s, int& mo, int& so) {
    const bool cand = lane_theta < __builtin_inf();
    const double nu = lane < 32 ? nu0 : nu1;
    const int c = lane & 31;
    int key;
    if (p.force_s >= 0) {
        key = row16_min_i((cand && ldexp(nu, -p.force_s) <= lane_theta) ? c : 1 << 20);
    } else {
        const int q = min(min_squarings(nu, cand ? lane_theta : 1.0), 63);
        key = row16_min_i(cand ? ((taylor_products(cand_degree(c)) + q) << 12) | (q << 5) | c : 0x7fffffff);
    }
    auto plan = [&](int k, int& mm, int& ss) {
        if (p.force_s >= 0) {
            mm = k < kNumCand ? cand_degree(k) : p.max_degree;
            ss = p.force_s;
        } else {
            mm = cand_degree(k & 31);
            ss = (k >> 5) & 63;
        }
    };
    plan(__builtin_amdgcn_readlane(key, 32 * team), m, s);
    plan(__builtin_amdgcn_readlane(key, 32 * (team ^ 1)), mo, so);
}

// The chain [j0, j1); its product is left in Q.  RT: the row tiles that the
// embedded dimension reaches.  OUT: with per-slice output (its addresses take
// registers that the other instances need for the products).
template <int PMODE, int RT, bool OUT>
__device__ __forceinline__ void panel_run(const PropParams& p, int64_t j0, int64_t j1, char* lds, PLane L,
                                          Tile<double> (&Q)[2]) {
    double* red = reinterpret_cast<double*>(lds + 4 * kPanelSlot);   // [parity][slice][half][row]
    double* wts = red + 2 * 2 * 2 * kPanelD;                          // [slice mod kPanelAhead][basis matrix]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            Q[i].re[r] = 32 * L.team + 16 * i + 4 * L.g + r == 16 * L.w + L.j ? 1.0 : 0.0;
            Q[i].im[r] = 0.0;
        }
    const int64_t jlast = p.n_slices > 0 ? p.n_slices - 1 : 0;
    const double lth = lane_theta_of(p, L.lane & 31);
    PanelExpand X;
    // Stage both slices' exponents, as they are: the scaling by 2^-s follows in the
    // products (exact), so the bound that s comes from and G share a barrier.
    auto stage_g = [&](char* sa, char* sb, int par) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) panel_stage_tile<PMODE>(t ? sb : sa, X.G[t][kk], 2 * L.team + kk, L);
            double rs = X.rs[t];
            rs += __shfl_xor(rs, 16);
            rs += __shfl_xor(rs, 32);
            if (L.g == 0) red[((par * 2 + t) * 2 + L.team) * kPanelD + 16 * L.w + L.j] = rs;
        }
    };
    auto bound = [&](int par, int t) {
        const double* v = red + (par * 2 + t) * 2 * kPanelD + L.lane;
        return wave_uniform(rows_max(row16_max(v[0] + v[kPanelD])));
    };
    // Slot roles: G (then the sine series, then a chain exchange) in u[slice], Y
    // (then E) in u[2 + slice].  After the last chain product of a pair slots 0
    // and 2 have no reader left while 1 and 3 (the exchange and E) may still
    // have one: slots 1 and 2 trade places for the next pair.
    char* u[4] = {lds, lds + kPanelSlot, lds + 2 * kPanelSlot, lds + 3 * kPanelSlot};
    // Weights of the slices j .. j + kPanelAhead - 1 (zero past the chain), all waves
    // at once: the samples come from HBM, and a prefetch in registers would need
    // more of them than there are.
    auto weights = [&](int64_t j) {
        for (int i = threadIdx.x; i < kPanelAhead * p.M; i += 512) {
            const int64_t js = j + i / p.M;
            const WeightRecipe wr = weight_recipe(p, i % p.M);
            wts[i] = js < j1 ? combine_weight(p, wr, gather_samples(p, wr, min(js, jlast))) : 0.0;
        }
    };
    __syncthreads();   // readers of what the block did before
    X.issue(p, 0, L);
    weights(j0);
    __syncthreads();
    X.rs[0] = X.rs[1] = 0.0;
    X.consume(p, 0, wts, L);
    X.issue(p, 1, L);
    X.consume(p, 1, wts, L);
    stage_g(u[0], u[1], 0);
    int par = 0;
    for (int64_t j = j0; j < j1; j += 2, par ^= 1) {
        char* s0 = L.team ? u[1] : u[0];
        char* s1 = L.team ? u[3] : u[2];
        L = fresh(L);
        __syncthreads();
        int m, s, mo, so;
        panel_plan(p, bound(par, 0), bound(par, 1), L.lane, lth, L.team, m, s, mo, so);
        const int next = (int)((j + 2 - j0) % kPanelAhead);   // the next pair's place in the table
        if (next == 0) weights(j + 2);
        const int mm = max(m, mo), rounds = wave_uniform(max(s, so));
        const bool low = min(m, mo) <= 2;
        if (low) {
            // degrees 1 and 2 need G itself in the panel layout: its halves are
            // exchanged in FP32
            f4_t* v0 = reinterpret_cast<f4_t*>(u[2]) + (L.w * 4 * 64 + L.lane) * 2;
            f4_t* v1 = reinterpret_cast<f4_t*>(u[3]) + (L.w * 4 * 64 + L.lane) * 2;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int at = (2 * L.team + kk) * 128;
                const Tile<float>&a = X.G[0][kk], &b = X.G[1][kk];
                v0[at] = f4_t{a.re[0], a.re[1], a.re[2], a.re[3]};
                v0[at + 1] = f4_t{a.im[0], a.im[1], a.im[2], a.im[3]};
                v1[at] = f4_t{b.re[0], b.re[1], b.re[2], b.re[3]};
                v1[at + 1] = f4_t{b.im[0], b.im[1], b.im[2], b.im[3]};
            }
            __syncthreads();
        }
        // The barriers of the two teams' branches pair up: one each for the
        // exchange, Y and the sine series, as far as either team needs them.
        Panel C;
        if (m >= 4) {
            panel_series<PMODE, RT>(m, s, low, s0, s1, L, C);
        } else {
            panel_short_series<PMODE, RT>(m, s, mm, low, s0, s1, L, C);
        }
        // C is E now
        if (rounds > 0) {
            panel_square(C, s, rounds, lds, L);
            panel_stage<PMODE>(s1, C, L);
        }
        L = fresh(L);
        if (OUT && j + L.team < j1) panel_store_slice(p, j + L.team, C, L);
        X.issue(p, 0, L);
        __syncthreads();
        X.rs[0] = X.rs[1] = 0.0;
        panel_chain<PMODE, RT>(Q, u[2], u[0], L);
        X.consume(p, 0, wts + next * p.M, L);
        if (j + 1 >= j1) break;
        X.issue(p, 1, L);
        L = fresh(L);
        panel_chain<PMODE, RT>(Q, u[3], u[1], L);
        X.consume(p, 1, wts + next * p.M, L);
        char* x = u[1];
        u[1] = u[2];
        u[2] = x;
        stage_g(u[0], u[1], par ^ 1);
    }
}

// Q into the strips of the product tree (waves 0..3: column strip c), through LDS.
__device__ __forceinline__ Strip<4> panel_to_strips(const Tile<double> (&Q)[2], char* lds, const PLane& L) {
    d2_t* s = reinterpret_cast<d2_t*>(lds);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            s[(32 * L.team + 16 * i + 4 * L.g + r) * kPanelRootLd + 16 * L.w + L.j] = d2_t{Q[i].re[r], Q[i].im[r]};
    __syncthreads();
    Strip<4> X;
    strip_each<4>([&](int k, int r) {
        const d2_t v = s[(16 * k + L.g + 4 * r) * kPanelRootLd + 16 * L.w + L.j];
        X.t[k].re[r] = v.x;
        X.t[k].im[r] = v.y;
    });
    __syncthreads();
    return X;
}

__device__ __forceinline__ PLane panel_lane() {
    PLane L;
    L.lane = threadIdx.x & 63;
    L.g = L.lane >> 4;
    L.j = L.lane & 15;
    const int wave = wave_uniform((int)(threadIdx.x >> 6));
    L.team = wave >> 2;
    L.w = wave & 3;
    return L;
}

}  // namespace
}  // namespace pm
