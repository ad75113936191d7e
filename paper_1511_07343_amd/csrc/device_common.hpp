// Device helpers shared by the correlation kernels (FFT and matrix forms).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace fdas {

constexpr double kLn2 = 0.69314718055994530942;

// m(k): block medians joined linearly between block centres, flat outside.
// Bin numbers fit 32 bits (a spectrum has at most 2^25 bins), whose
// conversions to and from FP64 are single instructions; no branches, so that
// the loads of several bins are in flight together.
__device__ __forceinline__ double median_curve(const double *__restrict__ med, int64_t nblk, int W,
                                               int64_t nb, int64_t g) {
    const int last = int(nblk) - 1;
    const double c0 = 0.5 * double(min(W, int(nb)) - 1);
    const int w0 = last * W;  // first bin of the last block
    const double cl = double(w0) + 0.5 * double(int(nb) - w0 - 1);
    const double x = double(int(g));
    // W is a power of two, so dividing by it is the exact multiply by 1 / W;
    // the last interval (to the centre of a partial last block) is shorter,
    // and its reciprocal width does not depend on g (computed once per
    // thread when inlined in a loop)
    const double inv_w = 1.0 / double(W);
    const double inv_last = 1.0 / (cl - (c0 + double(last - 1) * double(W)));
    const int b = max(0, min(int(floor((x - c0) * inv_w)), last - 1));
    const double lo = med[b], hi = med[min(b + 1, last)];
    const double cb = c0 + double(b) * double(W);
    const double f = (x - cb) * (b + 1 == last ? inv_last : inv_w);
    double mid = lo + (hi - lo) * f;
    asm("" : "+v"(mid));  // selected, not formed behind a branch that the loads are waited for at
    return x <= c0 ? lo : x >= cl ? hi : mid;
}

// The normalising factor sqrt(ln 2 / m) in FP64 (0 where m is not positive, or
// infinite): the hardware's reciprocal square root and two Newton steps, to a
// rounding or two of the division and square root, which take three times as
// long.  m lies between medians of single-precision powers, well inside the
// range of the steps; no branches, as above.
__device__ __forceinline__ double norm_scale(double m) {
    double r = __builtin_amdgcn_rsq(m);
    r = fma(0.5 * r, fma(-m * r, r, 1.0), r);
    r = fma(0.5 * r, fma(-m * r, r, 1.0), r);
    r *= 0.83255461115769775635;  // sqrt(ln 2)
    asm("" : "+v"(r));
    return m > 0.0 && m < __builtin_inf() ? r : 0.0;
}

// Screening code of a power: P / delta, code_inv = 1 / delta, rounded up, at
// most 255, so integer sums of codes bound power sums from above (up to one
// FP32 rounding of the sum below, which the thresholds in code units leave room
// for); NaN and huge powers saturate at 255 (the minimum drops a NaN).  The
// conversion rounds to the nearest integer, hence the half: with a whole unit
// the codes come out half a unit high, and the screen passes 28 % more cells
// on at 3 sigma, 16 harmonics (762078 against 597532 of 2^18 columns x 21
// templates).  Inserted as byte `b` of w: three instructions a code.
__device__ __forceinline__ uint32_t put_code(float pw, float code_inv, int b, uint32_t w) {
    return __builtin_amdgcn_cvt_pk_u8_f32(fminf(fmaf(pw, code_inv, 0.5f), 255.f), uint32_t(b), w);
}

// exp(-2 pi i k / 2M), which separates the spectrum of a real series of 2M
// samples from the M-point DFT of its even and odd samples, and its rotation
// by a step of bins (real_factor_step); FP64.
struct RealFactor {
    double c, s;
    __device__ __forceinline__ RealFactor(int64_t k, int64_t M) { sincospi(-double(k) / double(M), &s, &c); }
    __device__ __forceinline__ void rotate(double2 step) {
        const double c1 = fma(c, step.x, -(s * step.y));
        s = fma(c, step.y, s * step.x);
        c = c1;
    }
};

inline double2 real_factor_step(int bins, int64_t M) {
    const double a = -3.14159265358979323846 * double(bins) / double(M);
    return make_double2(cos(a), sin(a));
}

// X[k] = E + exp(-2 pi i k / 2M) O of the real series' spectrum,
// E = (Z[k] + conj Z[M-k]) / 2, O = (Z[k] - conj Z[M-k]) / (2i), 0 < k < M.
__device__ __forceinline__ float2 unpack_bin(float2 zk, float2 zm, const RealFactor &f) {
    const float2 e = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
    const float2 o = make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x));
    const float c = float(f.c), s = float(f.s);
    return make_float2(e.x + fmaf(o.x, c, -(o.y * s)), e.y + fmaf(o.x, s, o.y * c));  // as cmul
}

// The larger power of a 2-bin block, a NaN if either is one: powers are
// non-negative (or NaN), and non-negative floats, with NaN above +inf, order
// as their unsigned bit patterns, so one integer maximum picks the larger
// power and keeps a NaN (fmaxf alone would drop it).
__device__ __forceinline__ float block_power(float a, float b) {
    return __uint_as_float(max(__float_as_uint(a), __float_as_uint(b)));
}

// The codes of the two 2-bin blocks of 4 consecutive bins, as 2 bytes.
__device__ __forceinline__ uint16_t block_codes4(float4 p, float code_inv) {
    return uint16_t(put_code(block_power(p.z, p.w), code_inv, 1, put_code(block_power(p.x, p.y), code_inv, 0, 0u)));
}

// Single-trial significance in FP64: log Q(n, s) of a sum of n unit-mean
// exponential powers (n <= 16), and sigma with Phi_c(sigma) = Q(n, s).

// Q(n, s) = exp(-s) sum_{i < n} s^i / i!, the sum as 1 + s (1 + s/2 (1 + ...)).
__device__ inline double log_gamma_survival_d(int n, double s) {
    if (s <= 0.0) return 0.0;
    if (s > 1e18) return -s;  // the logarithm of the sum is below a rounding of s
    double sum = 1.0;
#pragma unroll
    for (int i = 15; i >= 1; --i)
        if (i < n) sum = fma(sum * s, 1.0 / double(i), 1.0);
    return log(sum) - s;
}

__device__ inline double log_normal_tail_d(double sg) { return log(0.5 * erfc(sg * 0.70710678118654752440)); }

// sigma <= 0: Newton's method inside a bracket that falls back to bisection
// whenever a step leaves it.
__device__ inline double significance_low_d(double target) {
    double lo = -40.0, hi = 1.0, x = 0.0;
    for (int it = 0; it < 100; ++it) {
        const double lt = log_normal_tail_d(x);
        const double f = lt - target;
        if (f > 0.0) lo = x; else hi = x;
        const double dlog = -exp(-0.5 * x * x - 0.91893853320467274178 - lt);  // d/dx log Phi_c
        double nx = x - f / dlog;
        if (fabs(nx - x) <= 1e-12 * fmax(1.0, fabs(x))) return nx;
        if (!(nx > lo && nx < hi)) nx = 0.5 * (lo + hi);
        x = nx;
        if (hi - lo <= 1e-12 * fmax(1.0, fabs(hi))) break;
    }
    return x;
}

// With E(x) = erfcx(x / sqrt 2): log Phi_c(x) = log(E / 2) - x^2 / 2 and its
// derivative -sqrt(2 / pi) / E.  log Phi_c is concave and decreasing, so after
// its first step Newton's method approaches the root from the right, and a
// step below 1e-7 leaves an error of its square.
__device__ inline double significance_d(double power, int n) {
    const double target = log_gamma_survival_d(n, power);
    if (!(target < -0.69314718055994530942)) return significance_low_d(target);
    constexpr double kMost = 1342177280.0;  // reported from there on (powers past 9e17, infinite ones)
    if (!(target > -0.5 * kMost * kMost)) return kMost;
    const double t = -2.0 * target;
    double x = sqrt(fmax(t - log(6.28318530717958647693 * t), 0.25));  // the tail's asymptote
    for (int it = 0; it < 50; ++it) {
        const double e = erfcx(x * 0.70710678118654752440);
        const double f = log(0.5 * e) - 0.5 * x * x - target;
        const double dx = f * e * 1.25331413731550025121;  // sqrt(pi / 2)
        x += dx;
        if (fabs(dx) <= 1e-7 * fmax(1.0, x)) break;
    }
    return x;
}

}  // namespace fdas
