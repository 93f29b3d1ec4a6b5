// Bounds of the basis matrices' 2-norms above 16 levels (FP64 contexts), formed
// where the basis already is.  On the host a matrix of 64 levels takes 150 us and
// one of 32 levels 30 us; here all of them take 41 and 24 us with launch and wait.
// (Up to 16 levels the host's 3 us a matrix are less: norm_bound.cpp.)
#include "mfma_strip.h"

namespace pm {
namespace {

// Upper bound of ||A||_2 of a Hermitian A: (||A^n||_F)^(1/n), n = 2^squarings by
// repeated squaring of the scaled matrix, never above ||A||_1.  It is within
// d^(1/2n) of the 2-norm (n = 16: 9 % at d = 16, n = 8: 30 % at d = 64, a third of that
// for a GUE matrix).  One strip team per matrix; bounds[m] comes in as ||B_m||_1.
template <int NT>
__global__ void __launch_bounds__(64 * NT) norm2_bounds(const double* basis, double* bounds, int squarings) {
    constexpr int D = 16 * NT;
    extern __shared__ char bsm[];
    constexpr size_t SB = strip_slot_bytes<NT>();
    Slots sl{{bsm, bsm + SB}, 0};
    double* red = reinterpret_cast<double*>(bsm + 2 * SB);
    SLane L;
    L.lane = threadIdx.x & 63;
    L.g = L.lane >> 4;
    L.j = L.lane & 15;
    L.c = wave_uniform((int)(threadIdx.x >> 6));
    const int m = blockIdx.x;
    const double n1 = bounds[m];
    if (!(n1 > 0.0)) {
        if (threadIdx.x == 0) bounds[m] = 0.0;
        return;   // the whole block
    }
    Strip<NT> A;
    const double inv = 1.0 / n1;
    strip_each<NT>([&](int k, int r) {
        A.t[k].re[r] = basis[mfma_basis_index(D, m, k, L.c, 0, r, L.lane)] * inv;
        A.t[k].im[r] = basis[mfma_basis_index(D, m, k, L.c, 1, r, L.lane)] * inv;
    });
    double lg = 0.0, bound = n1;   // lg: log ||(A / n1)^n||_F
    bool ok = true;
    for (int s = 0; s < squarings && ok; ++s) {
        A = strip_mul<NT, 4 * NT>(strip_put<NT>(sl, A, L), A, L);
        double f = 0.0;
        strip_each<NT>([&](int k, int r) { f = fma(A.t[k].re[r], A.t[k].re[r], fma(A.t[k].im[r], A.t[k].im[r], f)); });
#pragma unroll
        for (int x = 1; x < 64; x <<= 1) f += __shfl_xor(f, x);
        __syncthreads();
        if (L.lane == 0) red[L.c] = f;
        __syncthreads();
        f = 0.0;
#pragma unroll
        for (int c = 0; c < NT; ++c) f += red[c];
        f = sqrt(f);
        ok = f > 0.0;   // (the same sum in every wave)
        if (!ok) break;
        lg = 2.0 * lg + log(f);
        const double sc = 1.0 / f;
        strip_each<NT>([&](int k, int r) {
            A.t[k].re[r] *= sc;
            A.t[k].im[r] *= sc;
        });
    }
    if (ok) bound = fmin(n1, n1 * exp(lg / (double)(1 << squarings)));
    if (threadIdx.x == 0) bounds[m] = bound * (1.0 + 1e-6);
}

template <int NT>
hipError_t launch_bounds_t(const double* basis, double* bounds, int n, int squarings, hipStream_t stream) {
    constexpr size_t lds = 2 * strip_slot_bytes<NT>() + 64;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)norm2_bounds<NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((norm2_bounds<NT>), dim3((unsigned)n), dim3(64 * NT), lds, stream, basis, bounds, squarings);
    return hipGetLastError();
}

}  // namespace

// The bounds of the first n matrices of an FP64 basis of D-wide tiles, in place
// of their 1-norms in `bounds`.
hipError_t launch_norm2_bounds(int D, const double* basis, double* bounds, int n, hipStream_t stream) {
    switch (D) {
        case 32: return launch_bounds_t<2>(basis, bounds, n, 4, stream);
        case 64: return launch_bounds_t<4>(basis, bounds, n, 3, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace pm
