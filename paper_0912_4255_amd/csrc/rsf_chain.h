// The interpolated timing chain shared by the resampler and the point search,
// and small device helpers of both.
//
// Over a run of consecutive resampled samples every slowly varying quantity (the
// delay d, the beam patterns and, for the gradient, dT/dtheta and the patterns'
// derivatives) is the quartic through five exact nodes at s = -p, -q, 0, q and p
// samples from the run's centre, near the Chebyshev points of |s| <= half (the
// run and the interpolation window around it).  Each quantity is a sum of
// circular motions, so with rate w and H = half dt the remainder is at most
// A (w H)^5 / 1920, A the amplitude.  chain_interpolates() admits the sampling
// intervals for which that is at most `delay` (s) for t_m and `beam` for a and b
// (rate 2 w_sid; FP32 resolves 6e-8 of them, but the FP64 antenna sums of the
// resampler show more), orbit_slow() the orbits for which it is at most `delay` for
// R (and 3e-11 relative for its derivatives).  What goes on in FP32 takes kDelayErr:
// at 100 Hz and 1e-11 s the phase is off by 6e-9 rad.
#pragma once

#include <math.h>

#include "rsf_device.h"

namespace rsf {

constexpr float kPiF = 3.14159265358979323846f;

constexpr double kDelayErr = 1e-11;

// H: half dt, in seconds
inline bool chain_interpolates(const EphDev& e, double H, double delay, double beam) {
    const double xo = 2.0 * kPi * fabs(e.inv_p_orb) * H, xs = 2.0 * kPi * fabs(e.inv_p_sid) * H;
    auto p5 = [](double x) { return x * x * x * x * x / 1920.0; };
    return fabs(e.au_c) * p5(xo) + fabs(e.re_c) * p5(xs) <= delay && p5(2.0 * xs) <= beam && xo <= 0.1;
}
__device__ __forceinline__ bool orbit_slow(const BinaryOrbit& b, double H, double delay) {
    const double x = 2.0 * kPi / b.p_orb * H;
    return x <= 0.035 && b.a_p * (x * x) * (x * x) * x <= delay * 1920.0;
}

template <typename RUN>
__device__ __forceinline__ double node_at(int i) {
    return i == 0 ? -RUN::p : i == 1 ? -RUN::q : i == 2 ? 0.0 : i == 3 ? RUN::q : RUN::p;
}

__device__ __forceinline__ double quartic(const double* c, double s) {
    return c[0] + s * (c[1] + s * (c[2] + s * (c[3] + s * c[4])));
}

// node values at -p, -q, 0, q, p to the quartic's coefficients
template <typename RUN>
__device__ __forceinline__ void to_quartic(double* c) {
    constexpr double p = RUN::p, q = RUN::q, ip2 = 1.0 / (p * p), iq2 = 1.0 / (q * q), idiff = 1.0 / (p * p - q * q);
    const double f0 = c[2];
    const double ep = (0.5 * (c[4] + c[0]) - f0) * ip2, eq = (0.5 * (c[3] + c[1]) - f0) * iq2;
    const double op = 0.5 * (c[4] - c[0]) * (1.0 / p), oq = 0.5 * (c[3] - c[1]) * (1.0 / q);
    const double c4 = (ep - eq) * idiff, c3 = (op - oq) * idiff;
    c[0] = f0;
    c[1] = op - c3 * (p * p);
    c[2] = ep - c4 * (p * p);
    c[3] = c3;
    c[4] = c4;
}

// The delay at detector samples, k d / dt (k = f_het dt: cycles), as a quartic
// in x = (detector sample) - u_c, u_c the centre node's position: through the
// nodes at x_i = s_i - (v_i - v_2), v = d / dt there, by divided differences.
template <typename RUN>
__device__ __forceinline__ void window_delay(const double* v, double k, double* out) {
    double x[5], c[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        x[i] = node_at<RUN>(i) - (v[i] - v[2]);
        c[i] = k * v[i];
    }
#pragma unroll
    for (int j = 1; j < 5; ++j)
#pragma unroll
        for (int i = 4; i >= j; --i) c[i] = (c[i] - c[i - 1]) / (x[i] - x[i - j]);
    double m[5] = {c[4], 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 3; j >= 0; --j) {
#pragma unroll
        for (int i = 4 - j; i > 0; --i) m[i] = m[i - 1] - x[j] * m[i];
        m[0] = c[j] - x[j] * m[0];
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) out[i] = m[i];
}

__device__ __forceinline__ bool in_gap(const int64_t* __restrict__ gaps, int n_gaps, int64_t j) {
    int lo = 0, hi = n_gaps - 1, best = -1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        if (gaps[2 * mid] <= j) {
            best = mid;
            lo = mid + 1;
        } else {
            hi = mid - 1;
        }
    }
    return best >= 0 && j < gaps[2 * best + 1];
}

// Where samples lo .. hi lie: 0 outside every gap, 1 inside one, 2 to be looked
// up one by one (in_gap).
__device__ __forceinline__ int gap_state(const int64_t* __restrict__ gaps, int n_gaps, int64_t lo, int64_t hi) {
    int b = -1;  // the last gap that starts at or before hi
    for (int l = 0, h = n_gaps - 1; l <= h;) {
        const int mid = (l + h) >> 1;
        if (gaps[2 * mid] <= hi) {
            b = mid;
            l = mid + 1;
        } else {
            h = mid - 1;
        }
    }
    if (b < 0 || gaps[2 * b + 1] <= lo) return 0;
    return gaps[2 * b] <= lo && gaps[2 * b + 1] > hi ? 1 : 2;
}

// sinc(x) = sin(pi x)/(pi x) and its derivative from accurate sin(pi x), cos(pi x);
// a series near 0 avoids the cancellation in (cos(pi x) - sinc(x)) / x.
__device__ __forceinline__ void sinc_d(float x, float sx, float cx, float& s, float& ds) {
    if (fabsf(x) < 0.05f) {
        const float p2 = kPiF * kPiF * x * x;
        s = 1.f - p2 / 6.f + p2 * p2 / 120.f - p2 * p2 * p2 / 5040.f;
        ds = -(kPiF * kPiF * x / 3.f) * (1.f - p2 / 10.f + p2 * p2 / 280.f);
    } else {
        const float rx = __builtin_amdgcn_rcpf(x);
        s = sx * rx * (1.f / kPiF);
        ds = (cx - s) * rx;
    }
}

}  // namespace rsf
