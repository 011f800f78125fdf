// rcmc_fit.hpp -- the RCMC weights and the plan's tables of them.
//
// The 8-tap Kaiser-windowed sinc (taps t = -3..4 about floor(p), x = p -
// floor(p), weights normalised to unit sum) depends on x alone.  Its eight
// weight functions w_t(x) are smooth on [0, 1), so the plan stores them as
// piecewise quadratics: RCMC_INTERVALS intervals, on each a degree-2
// Chebyshev interpolant of the exact FP64 weights, in monomial form in the
// local variable u = x * RCMC_INTERVALS - b in [0, 1].  Layout (interval-
// major, 24 floats = 96 bytes per interval, read as six 16-byte vectors):
//     tab[b * 24 + t * 3 + j] = coefficient of u^j, tap t.
// The interpolation error is 2.2e-8 in FP64 (below the FP32 rounding of the
// coefficients; tested against the oracle's weights).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace sar {

constexpr int RCMC_INTERVALS = 128;
constexpr int RCMC_PER_INTERVAL = 24;
constexpr int RCMC_TAB = RCMC_INTERVALS * RCMC_PER_INTERVAL;
// k_rcmc_rows evaluates the weights of four output rows on one interval, that of
// their middle, so up to RROWS_MARGIN of an interval beyond its ends.  Quadratics
// on the intervals above have 7.1e-8 there, so it has cubics of its own, on 48
// intervals and fitted over the margins too: 2.1e-9 (3.4e-9 at beta = 0), and with
// their FP32 coefficients 3.0e-8 to 4.5e-8 where the quadratics have 5.1e-8 to 7.1e-8
// within their intervals.  Three FMAs per weight instead of two: the 4096 x 4096
// hyperbolic scene takes 1% longer, 8192 x 4096 and half storage as long.
//     behind the quadratics: tab[RCMC_TAB + b * 32 + t * 4 + j]
constexpr double RCMC_ROWS_STRETCH_MAX = 5e-4;   // change of shift per row, cells
constexpr int RROWS_INTERVALS = 48;
constexpr int RROWS_PER_INTERVAL = 32;
constexpr int RROWS_TAB = RROWS_INTERVALS * RROWS_PER_INTERVAL;
constexpr double RROWS_MARGIN = 1.5 * RCMC_ROWS_STRETCH_MAX * RROWS_INTERVALS;   // half of three rows' change
// the outermost of four nodes, 0.5 + 0.9239 (0.5 + margin), stays within the interval:
// beyond [0, 1) a tap may leave the window, where its weight has a kink
static_assert(RROWS_MARGIN < 0.04, "nodes within the interval");

__host__ __device__ inline double sin_pi(double x)
{
#ifdef __HIP_DEVICE_COMPILE__
    return sinpi(x);
#else
    return std::sin(3.14159265358979323846 * x);
#endif
}
__host__ __device__ inline double cos_pi(double x)
{
#ifdef __HIP_DEVICE_COMPILE__
    return cospi(x);
#else
    return std::cos(3.14159265358979323846 * x);
#endif
}

__host__ __device__ inline double i0_fp64(double y)
{
    const double q = 0.25 * y * y;
    double term = 1.0, sum = 1.0;
    for (int k = 1; k < 200; ++k) {
        term *= q / ((double)k * (double)k);
        sum += term;
        if (term < 1e-17 * sum) break;
    }
    return sum;
}

// Exact normalised weights at x (FP64): K(z) = sinc(z) I0(beta sqrt(1-(z/4)^2)).
__host__ __device__ inline void kaiser_weights_fp64(double x, double beta, double* w)
{
    double sum = 0.0;
    for (int i = 0; i < 8; ++i) {
        const double z = (double)(i - 3) - x;
        const double r = z / 4.0;
        const double sc = (z == 0.0) ? 1.0 : sin_pi(z) / (3.14159265358979323846 * z);
        const double arg = 1.0 - r * r;
        w[i] = (arg > 0.0 ? sc * i0_fp64(beta * sqrt(arg)) : 0.0);
        sum += w[i];
    }
    for (int i = 0; i < 8; ++i) w[i] /= sum;
}

// Monomial coefficients in u of the degree-D interpolant of the weights on
// interval b of `intervals`: D + 1 Chebyshev nodes over [-margin, 1 + margin], exact
// weights, one linear solve per tap.
template <int D>
__host__ __device__ void rcmc_fit(float* __restrict__ out, int b, int intervals, double margin, double beta)
{
    constexpr int K = D + 1;
    double u[K], w[K][8];
    for (int j = 0; j < K; ++j) {
        u[j] = 0.5 * (1.0 + (1.0 + 2.0 * margin) * cos_pi((2.0 * j + 1.0) / (2.0 * K)));
        kaiser_weights_fp64(((double)b + u[j]) / intervals, beta, w[j]);
    }
    for (int t = 0; t < 8; ++t) {
        double M[K][K + 1];
        for (int j = 0; j < K; ++j) {
            M[j][0] = 1.0;
            for (int c = 1; c < K; ++c) M[j][c] = M[j][c - 1] * u[j];
            M[j][K] = w[j][t];
        }
        for (int c = 0; c < K; ++c) {             // Gaussian elimination, partial pivot
            int piv = c;
            for (int r = c + 1; r < K; ++r)
                if (fabs(M[r][c]) > fabs(M[piv][c])) piv = r;
            for (int q = 0; q <= K; ++q) { double tmp = M[c][q]; M[c][q] = M[piv][q]; M[piv][q] = tmp; }
            for (int r = c + 1; r < K; ++r) {
                const double f = M[r][c] / M[c][c];
                for (int q = c; q <= K; ++q) M[r][q] -= f * M[c][q];
            }
        }
        double cf[K];
        for (int c = D; c >= 0; --c) {
            double acc = M[c][K];
            for (int q = c + 1; q < K; ++q) acc -= M[c][q] * cf[q];
            cf[c] = acc / M[c][c];
        }
        for (int j = 0; j < K; ++j) out[t * K + j] = (float)cf[j];
    }
}

}  // namespace sar
