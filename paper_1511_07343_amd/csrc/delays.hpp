// Dispersion delays of the de-dispersion, formed on the device; compiled for
// the host too, where the bounds of delay_fast are tested.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>

namespace fdas {

constexpr int DD_LAUNCH_DMS = 256;  // DM trials per launch (passed by value)

// What the delays are formed from; kdm[i] is the dispersion constant times DM i.
struct Dispersion {
    double f_top, foff, inv_top2, tsamp, inv_tsamp;  // inv_top2 = 1 / f_top^2
    double kdm[DD_LAUNCH_DMS];
};

// f_c^2, f_c = f_top - c foff, each operation rounded by itself: fused, f_c
// would differ by a rounding of f_top, which is f_top / f_c roundings of its own.
__host__ __device__ __forceinline__ double squared_frequency(const Dispersion &p, int c) {
#pragma clang fp contract(off)
    const double f = p.f_top - p.foff * double(c);
    return f * f;
}

// Delay of channel c: floor(kdm (1 / f_c^2 - 1 / f_top^2) / tsamp + 1/2), each
// operation rounded by itself, the same on the host and the device.
__host__ __device__ inline int32_t delay_of(const Dispersion &p, double kdm, int c) {
#pragma clang fp contract(off)
    const double raw = kdm * (1.0 / squared_frequency(p, c) - p.inv_top2) / p.tsamp;
    return int32_t(floor(raw + 0.5));
}

// 1 / x to 24 bits or better.
__host__ __device__ __forceinline__ double short_reciprocal(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rcp(x);
#else
    double y = 1.0 / x;
    uint64_t bits;
    std::memcpy(&bits, &y, 8);
    if (std::isfinite(y)) bits &= ~((uint64_t(1) << 29) - 1);
    std::memcpy(&y, &bits, 8);
    return y;
#endif
}

// Whether any lane of the wave answers yes (on the host: this one).
__host__ __device__ __forceinline__ bool any_lane(bool yes) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __any(yes);
#else
    return yes;
#endif
}

// The same without its divisions, which take most of its time: of the same
// f^2, two Newton steps on its reciprocal and a product with 1 / tsamp differ
// from the rounded operations by less than 2^-46 of kdm / (f^2 tsamp) (2^-1016
// of kdm / tsamp where 1 / f^2 is not a normal number).  A sum closer than
// that to a whole number (as with DM 0) is formed by delay_of, and so is one
// for which the comparison fails: factors may overflow though the delay is 0.
__host__ __device__ __forceinline__ int32_t delay_fast(const Dispersion &p, double kdm, int c) {
    const double f2 = squared_frequency(p, c);
    double y = short_reciprocal(f2);
    y = fma(fma(-f2, y, 1.0), y, y);
    y = fma(fma(-f2, y, 1.0), y, y);
    const double scale = kdm * p.inv_tsamp;
    const double x = fma(scale, y - p.inv_top2, 0.5);
    const double fl = floor(x), off = x - fl;
    const double slack = scale * (y + 0x1p-970) * 0x1p-46 + 0x1p-46;
    int32_t d = 0;
    if (any_lane(!(off >= slack && off <= 1.0 - slack))) d = delay_of(p, kdm, c);
    else d = int32_t(fl);
    return d;
}

}  // namespace fdas
