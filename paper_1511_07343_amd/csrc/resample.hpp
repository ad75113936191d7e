// Sample positions of the time-domain search; compiled for the host too, where
// their error is tested.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace fdas {

// 1 / sqrt(x) and 1 / x to about 22 bits.
__host__ __device__ __forceinline__ float short_rsqrt(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rsqf(x);
#else
    return 1.f / std::sqrt(x);
#endif
}
__host__ __device__ __forceinline__ float short_rcp(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rcpf(x);
#else
    return 1.f / x;
#endif
}

// Sample m of the series resampled for drift alpha lies at s_m = N (v_m + 1/2),
// v_m + alpha v_m^2 / 2 = tau_m = m / N - 1/2, the time axis on which a tone
// drifting by alpha (relative to its mean frequency) keeps one frequency.  The
// position is formed in FP64 (it needs ~24 bits of integer part plus the
// fraction): two Newton steps from the FP32 root v = 2 tau / (1 + sqrt(q)),
// q = 1 + 2 alpha tau in [1/2, 3/2], whose slope 1 + alpha v is sqrt(q), so no
// FP64 root or division is taken; the first leaves about 1e-14, the second a
// rounding.
struct DriftPositions {
    double h, inv_n;  // alpha / 2, 1 / N (exact: N is a power of two)

    __host__ __device__ __forceinline__ double newton(double v, double inv, double tau) const {
        return fma(tau - v * fma(h, v, 1.0), inv, v);
    }
    // v of samples 2 i and 2 i + 1.
    __host__ __device__ __forceinline__ void pair(int64_t i, double &v, double &w) const {
        const double tau0 = fma(double(int(2 * i)), inv_n, -0.5), tau1 = tau0 + inv_n;  // exact
        const float tf = float(tau0);
        const float q = fmaf(4.f * float(h), tf, 1.f);
        const float r = short_rsqrt(q);
        const double inv = double(r);
        v = double(2.f * tf * short_rcp(fmaf(q, r, 1.f)));
        v = newton(newton(v, inv, tau0), inv, tau0);
        w = fma(inv_n, inv, v);
        // 1 / sqrt(q) of the second sample, to first order in the step of q: with
        // the first's, short series of large drifts keep 1e-13
        const double inv1 = double(r * fmaf(-2.f * float(h) * float(inv_n) * r, r, 1.f));
        w = newton(newton(w, inv1, tau1), inv1, tau1);
    }
};

}  // namespace fdas
