// Time-domain resampling acceleration search (the other method of Sec. 1:
// resample the series for each acceleration trial, then one long DFT each).
// The DFT, the block medians and the harmonic sums are the FDAS kernels; this
// file holds the resampling and the normalised powers with their screening
// codes.
#include "device_common.hpp"
#include "kernels.hpp"

#include <cmath>

namespace fdas {

namespace {

// y[m] = x at position s_m = N (v_m + 1/2), v_m = 2 tau_m / (1 + sqrt(1 + 2 alpha tau_m)),
// tau_m = m / N - 1/2: the time axis on which a tone drifting by alpha
// (relative to its mean frequency) keeps one frequency.  Linear interpolation
// between the neighbouring samples (x[N] = 0), zero outside the series.  The
// position is formed in FP64 (it needs ~24 bits of integer part plus the
// fraction); its square root and division, most of the kernel's instructions
// when done by the library, start from the hardware's approximations and take
// two Newton steps each (arguments in [1/2, 3/2] and [1, 3]).
__device__ __forceinline__ float resampled(const float *__restrict__ x, int n, double nd, double alpha, double tau) {
    const double q = fma(2.0 * alpha, tau, 1.0);
    double r = __builtin_amdgcn_rsq(q);
    r = fma(0.5 * r, fma(-q * r, r, 1.0), r);
    r = fma(0.5 * r, fma(-q * r, r, 1.0), r);
    const double d = fma(q, r, 1.0);  // 1 + sqrt(q)
    double inv = __builtin_amdgcn_rcp(d);
    inv = fma(fma(-d, inv, 1.0), inv, inv);
    inv = fma(fma(-d, inv, 1.0), inv, inv);
    const double s = nd * fma(2.0 * tau, inv, 0.5);
    const double fl = floor(s);
    const int i = int(fl);
    if (!(i >= 0 && i <= n - 1)) return 0.f;
    const double f = s - fl;
    const double a = double(x[i]);
    const double b = i + 1 < n ? double(x[i + 1]) : 0.0;
    return float(a * (1.0 - f) + b * f);
}

// Two trials' worth of launches at 2^23 samples or sixteen at 2^20 go together
// (blockIdx.y), four consecutive samples per thread.  n % 1024 == 0.
__global__ __launch_bounds__(256) void k_td_resample(const float *__restrict__ x, int n, double zmax, double dz, int nz,
                                                     int iz0, float *__restrict__ y) {
    double alpha;
    {
        // -alpha_max + d iz with two roundings, as the trials are defined
#pragma clang fp contract(off)
        alpha = nz == 1 ? 0.0 : -zmax + dz * double(iz0 + int(blockIdx.y));
    }
    const int m = 4 * (int(blockIdx.x) * 256 + int(threadIdx.x));
    const double nd = double(n), inv_n = 1.0 / nd;  // exact: n is a power of two
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = resampled(x, n, nd, alpha, double(m + j) * inv_n - 0.5);
    *reinterpret_cast<float4 *>(y + int64_t(blockIdx.y) * n + m) = make_float4(v[0], v[1], v[2], v[3]);
}

// P[k] = |X[k]|^2 ln2 / m(k) for 4 consecutive bins per thread, and the
// screening codes of their two 2-bin blocks.  nb % 4 == 0.
__global__ __launch_bounds__(256) void k_td_power(const float2 *__restrict__ X, const double *__restrict__ med, int W,
                                                  int64_t nb, int iz0, float *__restrict__ plane,
                                                  uint8_t *__restrict__ codes, float code_inv) {
    const int64_t c = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (4 * c >= nb) return;
    const int64_t nblk = (nb + W - 1) / W;
    const int64_t row = iz0 + int64_t(blockIdx.y);
    X += int64_t(blockIdx.y) * nb + 4 * c;
    med += int64_t(blockIdx.y) * nblk;
    const float4 v01 = reinterpret_cast<const float4 *>(X)[0], v23 = reinterpret_cast<const float4 *>(X)[1];
    const float re[4] = {v01.x, v01.z, v23.x, v23.z}, im[4] = {v01.y, v01.w, v23.y, v23.w};
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double m = median_curve(med, nblk, W, nb, 4 * c + i);
        const double scale = m > 0.0 ? kLn2 / m : 0.0;
        p[i] = float((double(re[i]) * double(re[i]) + double(im[i]) * double(im[i])) * scale);
    }
    const float4 p4 = make_float4(p[0], p[1], p[2], p[3]);
    *reinterpret_cast<float4 *>(plane + row * nb + 4 * c) = p4;
    *reinterpret_cast<uint16_t *>(codes + row * (nb / 2) + 2 * c) = block_codes4(p4, code_inv);
}

}  // namespace

hipError_t launch_td_resample(const float *x, int64_t nsamp, double zmax, double dz, int nz, int iz0, int count,
                              float *y, hipStream_t st) {
    if (nsamp <= 0 || nsamp % 1024 != 0 || nsamp > (int64_t(1) << 26) || count < 1 || count > 65535)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_td_resample, dim3(unsigned(nsamp / 1024), unsigned(count)), dim3(256), 0, st, x, int(nsamp),
                       zmax, dz, nz, iz0, y);
    return hipGetLastError();
}

hipError_t launch_td_power(const float2 *X, const double *med, int W, int64_t nb, int iz0, int count, float *plane,
                           uint8_t *codes, float code_inv, hipStream_t st) {
    if (nb <= 0 || nb % 4 != 0 || W <= 0 || count < 1 || count > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_td_power, dim3(unsigned((nb / 4 + 255) / 256), unsigned(count)), dim3(256), 0, st, X, med, W, nb,
                       iz0, plane, codes, code_inv);
    return hipGetLastError();
}

}  // namespace fdas
