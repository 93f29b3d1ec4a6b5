// Bounds of the basis matrices' 2-norms up to 16 levels (FP64 contexts).
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstring>

namespace pm {
namespace {

// One squaring of a Hermitian matrix of up to 16 levels, padded with zeros to 16
// (n: its levels up to a multiple of two), and the square of the result's Frobenius norm.
// Full rows in whole vectors: the baseline instruction set takes 2.1 us for 16
// levels with the lower triangle mirrored, AVX2 0.9 us without.
struct Square16 {
    alignas(32) double re[16 * 16], im[16 * 16];
};
typedef double V4 __attribute__((ext_vector_type(4)));

inline __attribute__((always_inline)) double square_rows(const Square16& x, Square16& y, int n) {
    V4 f = {};
    for (int i = 0; i < n; i += 2)
        for (int j = 0; j < n; j += 8) {
            V4 re[2][2] = {}, im[2][2] = {};
            for (int q = 0; q < n; ++q) {
                const V4* br = reinterpret_cast<const V4*>(x.re + 16 * q + j);
                const V4* bi = reinterpret_cast<const V4*>(x.im + 16 * q + j);
                for (int a = 0; a < 2; ++a) {
                    const double ar = x.re[16 * (i + a) + q], ai = x.im[16 * (i + a) + q];
                    for (int b = 0; b < 2; ++b) {
                        re[a][b] += ar * br[b];
                        re[a][b] -= ai * bi[b];
                        im[a][b] += ar * bi[b];
                        im[a][b] += ai * br[b];
                    }
                }
            }
            for (int a = 0; a < 2; ++a)
                for (int b = 0; b < 2; ++b) {
                    *reinterpret_cast<V4*>(y.re + 16 * (i + a) + j + 4 * b) = re[a][b];
                    *reinterpret_cast<V4*>(y.im + 16 * (i + a) + j + 4 * b) = im[a][b];
                    f += re[a][b] * re[a][b] + im[a][b] * im[a][b];
                }
        }
    return (f[0] + f[1]) + (f[2] + f[3]);
}

#if defined(__HIP_DEVICE_COMPILE__)
double square_avx2(const Square16& x, Square16& y, int n) { return square_rows(x, y, n); }
#else
__attribute__((target("avx2,fma"))) double square_avx2(const Square16& x, Square16& y, int n) { return square_rows(x, y, n); }
#endif
double square_base(const Square16& x, Square16& y, int n) { return square_rows(x, y, n); }

}  // namespace

// Upper bound of ||A||_2 of a Hermitian A of up to 16 levels from its 1-norm n1:
// (||A^16||_F)^(1/16) by repeated squaring of the scaled matrix, never above n1.  It
// is within d^(1/32) of the 2-norm (9 % at d = 16, a third of that for a GUE matrix).
// (More levels: engine_bounds.hip.)
double norm2_bound(const std::complex<double>* a, int d, double n1) {
    if (!(n1 > 0.0)) return 0.0;
    static const bool avx2 = __builtin_cpu_supports("avx2") && __builtin_cpu_supports("fma");
    Square16 m[2];
    std::memset(&m[0], 0, sizeof(m[0]));
    for (int r = 0; r < d; ++r)
        for (int c = 0; c < d; ++c) {
            m[0].re[16 * r + c] = a[r * d + c].real() / n1;
            m[0].im[16 * r + c] = a[r * d + c].imag() / n1;
        }
    double lg = 0.0;   // log ||(A / n1)^n||_F
    for (int k = 0; k < 4; ++k) {
        const Square16& x = m[k & 1];
        Square16& y = m[(k + 1) & 1];
        const int n = (d + 1) / 2 * 2;
        // (columns past n, up to the vector's end, are sums of zeros; rows past n are not read)
        const double f = std::sqrt(avx2 ? square_avx2(x, y, n) : square_base(x, y, n));
        if (!(f > 0.0)) return n1 * (1.0 + 1e-6);
        lg = 2.0 * lg + std::log(f);
        const double inv = 1.0 / f;
        for (int r = 0; r < n; ++r)
            for (int c = 0; c < n; ++c) {
                y.re[16 * r + c] *= inv;
                y.im[16 * r + c] *= inv;
            }
    }
    return std::min(n1, n1 * std::exp(lg / 16)) * (1.0 + 1e-6);
}

}  // namespace pm
