// Time-domain resampling acceleration search (the other method of Sec. 1:
// resample the series for each acceleration trial, then one long DFT each).
// The DFT (whose first pass resamples), the block medians and the harmonic sums
// are the FDAS kernels; this file holds the normalised powers with their
// screening codes.
#include "device_common.hpp"
#include "kernels.hpp"

#include <cmath>

namespace fdas {

namespace {

// |X|^2 ln2 / m for the median curve's value m: the hardware's reciprocal and
// two Newton steps (medians are single floats or their means, never FP64
// denormals; an infinite one gives 0).
__device__ __forceinline__ float normalised_power(float2 x, double m) {
    double r = __builtin_amdgcn_rcp(m);
    r = fma(fma(-m, r, 1.0), r, r);
    r = fma(fma(-m, r, 1.0), r, r);
    const double scale = m > 0.0 && m < INFINITY ? kLn2 * r : 0.0;
    return float((double(x.x) * double(x.x) + double(x.y) * double(x.y)) * scale);
}

// P[k] = |X[k]|^2 ln2 / m(k) and the screening codes of the 2-bin blocks, X
// unpacked from Z (a second time, after the median pass: X is neither written
// nor read).  A thread takes bins k .. k + 3 of the lower half and the four
// that mirror k + 1 .. k + 4: they need the same points of Z and, but for a
// sign, the same factors.  Sixteen spectra of 2^19 bins: 25 us (unpacked and
// stored by the median pass, 24 us here and 7 us more there).  nb % 8 == 0.
__global__ __launch_bounds__(256) void k_td_power(const float2 *__restrict__ Z, double2 step,
                                                  const double *__restrict__ med, int W, int64_t nb, int iz0,
                                                  float *__restrict__ plane, uint8_t *__restrict__ codes,
                                                  float code_inv) {
    const int64_t k0 = 4 * (int64_t(blockIdx.x) * 256 + threadIdx.x), h0 = nb - k0 - 4;
    if (2 * k0 >= nb) return;
    const int64_t nblk = (nb + W - 1) / W;
    const int64_t row = iz0 + int64_t(blockIdx.y);
    Z += int64_t(blockIdx.y) * nb;
    med += int64_t(blockIdx.y) * nblk;
    float2 lo[5], hi[5];  // Z[k0 + i], Z[nb - k0 - i]
    {
        const float4 a = reinterpret_cast<const float4 *>(Z + k0)[0], b = reinterpret_cast<const float4 *>(Z + k0)[1];
        const float4 c = reinterpret_cast<const float4 *>(Z + h0)[0], d = reinterpret_cast<const float4 *>(Z + h0)[1];
        lo[0] = make_float2(a.x, a.y);
        lo[1] = make_float2(a.z, a.w);
        lo[2] = make_float2(b.x, b.y);
        lo[3] = make_float2(b.z, b.w);
        lo[4] = Z[k0 + 4];
        hi[0] = k0 > 0 ? Z[nb - k0] : make_float2(0.f, 0.f);
        hi[1] = make_float2(d.z, d.w);
        hi[2] = make_float2(d.x, d.y);
        hi[3] = make_float2(c.z, c.w);
        hi[4] = make_float2(c.x, c.y);
    }
    RealFactor f(k0, nb);
    float p[4], q[4];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        if (i < 4) {
            const float2 x = i > 0 || k0 > 0 ? unpack_bin(lo[i], hi[i], f) : make_float2(0.f, 0.f);
            p[i] = normalised_power(x, median_curve(med, nblk, W, nb, k0 + i));
        }
        if (i > 0) {
            RealFactor g = f;  // bin nb - k: minus the conjugate
            g.c = -g.c;
            q[4 - i] = normalised_power(unpack_bin(hi[i], lo[i], g), median_curve(med, nblk, W, nb, nb - k0 - i));
        }
        f.rotate(step);
    }
    plane += row * nb;
    codes += row * (nb / 2);
    const float4 p4 = make_float4(p[0], p[1], p[2], p[3]), q4 = make_float4(q[0], q[1], q[2], q[3]);
    *reinterpret_cast<float4 *>(plane + k0) = p4;
    *reinterpret_cast<float4 *>(plane + h0) = q4;
    *reinterpret_cast<uint16_t *>(codes + k0 / 2) = block_codes4(p4, code_inv);
    *reinterpret_cast<uint16_t *>(codes + h0 / 2) = block_codes4(q4, code_inv);
}

}  // namespace

hipError_t launch_td_power(const float2 *Z, const double *med, int W, int64_t nb, int iz0, int count, float *plane,
                           uint8_t *codes, float code_inv, hipStream_t st) {
    if (nb <= 0 || nb % 8 != 0 || W <= 0 || count < 1 || count > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_td_power, dim3(unsigned((nb / 8 + 255) / 256), unsigned(count)), dim3(256), 0, st, Z,
                       real_factor_step(1, nb), med, W, nb, iz0, plane, codes, code_inv);
    return hipGetLastError();
}

}  // namespace fdas
