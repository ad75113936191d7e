// Fourier interpolation of the correlation off the (k, z) grid and the
// refinement of candidates by a pattern search over fractional (r, z).  This
// extends the paper's method: the drifting-tone response of Sec. 2 (the
// template of Eq. (1)) is evaluated at any offset and drift instead of the
// integer offsets of the template bank.  Everything is FP64 except the
// spectrum, which is read in FP32 as the search holds it.
#include "device_common.hpp"
#include "fresnel_coeffs.hpp"
#include "kernels.hpp"

#include <cmath>
#include <mutex>

namespace fdas {

namespace {

constexpr double kPiD = 3.14159265358979323846264338327950288;
// A workgroup refines one record at a time; its 16 waves share the record's
// (point, harmonic) pairs, so that a few hundred records fill the GPU.
constexpr int RF_THREADS = 1024;
constexpr int RF_POINT_THREADS = 256;  // workgroup of the point evaluator
constexpr int RF_POINTS = 8;    // neighbours per search level
constexpr int RF_MAX_NH = 16;

struct c64 {
    double re, im;
};
__device__ __forceinline__ c64 cadd(c64 a, c64 b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ c64 csub(c64 a, c64 b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ c64 cmul(c64 a, c64 b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ __forceinline__ c64 cscale(c64 a, double s) { return {a.re * s, a.im * s}; }
__device__ __forceinline__ double cnorm2(c64 a) { return a.re * a.re + a.im * a.im; }
// exp(i pi x), with x reduced to [0, 2) first and exact values at the
// multiples of 1/2 (so that integer offsets give exact results).
__device__ c64 cis_pi(double x) {
    const double r = x - 2.0 * floor(0.5 * x);
    if (r == 0.0) return {1.0, 0.0};
    if (r == 0.5) return {0.0, 1.0};
    if (r == 1.0) return {-1.0, 0.0};
    if (r == 1.5) return {0.0, -1.0};
    double s, c;
    sincospi(r, &s, &c);
    return {c, s};
}

// Fresnel integrals F(x) = C(x) + i S(x), C(x) = int_0^x cos(pi t^2 / 2) dt,
// from the polynomial data of fresnel_coeffs.hpp (written by
// gen_fresnel_coeffs.py): the auxiliary functions f, g of
// F(x) = (1 + i)/2 - (g + i f) exp(i pi x^2 / 2) on [0, 3) and [3, inf), and
// the power series of F for |x| < 1.  Horner's scheme with the coefficients
// read by uniform (scalar) loads; a range no lane of the wave needs is skipped.

// Two polynomials of N coefficients at t, {second, first}.  The address is
// made opaque at each use: the compiler would otherwise keep all coefficients
// across the caller's loops, far more than there are scalar registers.
template <int N>
__device__ __forceinline__ c64 poly_pair(const double (&c)[N][2], double t) {
    typedef const double __attribute__((address_space(4))) *Uniform;  // constant memory: scalar loads
    Uniform p = (Uniform)(uintptr_t)&c[0][0];
    asm volatile("" : "+s"(p));
    double a = p[2 * N - 2], b = p[2 * N - 1];
#pragma unroll
    for (int i = N - 2; i >= 0; --i) {
        a = fma(a, t, p[2 * i]);
        b = fma(b, t, p[2 * i + 1]);
    }
    return {b, a};
}

// G(x) = g(x) + i f(x) for x >= 0.
__device__ __forceinline__ c64 fresnel_aux(double x) {
    using namespace fresnel_data;
    c64 r = {0.0, 0.0};
    const bool far = x >= kSplit;
    if (__any(far)) {
        double inv = __builtin_amdgcn_rcp(x);
        inv = fma(fma(-x, inv, 1.0), inv, inv);
        inv = fma(fma(-x, inv, 1.0), inv, inv);
        const double u = inv * inv, t = fma(2.0 * kSplit * kSplit, u, -1.0);
        const c64 phi = poly_pair(kTail, t);
        const double ipx = inv * (1.0 / kPiD);  // f = phi_f / (pi x), g = phi_g / (pi^2 x^3)
        r = {phi.re * (u * ipx * (1.0 / kPiD)), phi.im * ipx};
    }
    if (!__all(far)) {
        const c64 near = poly_pair(kSmall, fma(x, 2.0 / kSplit, -1.0));
        r = far ? r : near;
    }
    return r;
}

// F(x) for |x| < 1: C = x sum c_n x^4n, S = x^3 sum s_n x^4n (Horner).
__device__ __forceinline__ c64 fresnel_small(double x) {
    using namespace fresnel_data;
    const double x2 = x * x, t = x2 * x2;
    const c64 p = poly_pair(kSeries, t);
    return {x * p.im, x * x2 * p.re};
}

// A(q, z) = int_0^1 exp(2 pi i [(q - z/2) u + z u^2 / 2]) du: the Fourier
// response at offset q bins of a unit tone whose frequency drifts by z bins
// over the observation (Sec. 2).  For z > 0, with p = q - z/2, Y = p sqrt(2/z),
// Z = Y + sqrt(2z) (so that pi (Z^2 - Y^2) / 2 = 2 pi q),
//   A sqrt(2z) = exp(-i pi Y^2 / 2) (F(Z) - F(Y)),
// and by the auxiliary functions, with e2q = exp(2 pi i q),
//   Y >= 0:      G(Y) - e2q G(Z)
//   Z < 0:       e2q G(-Z) - G(-Y)
//   Y < 0 <= Z:  (1 + i) exp(-i pi Y^2 / 2) - e2q G(Z) - G(-Y):
// one formula with the signs of Y and Z, whose exponential only the bins
// inside the drift need.  In waves that have such bins, the ones whose ends
// both lie within 1 of 0 (small z) take the difference of the power series,
// which does not cancel.  (With no bin inside, at most the nearest one cancels;
// it is nearly all of the response then, and its error that of a factor, which
// the power's normaliser takes out.)
// z < 0: conj(A(-q, -z)).  z = 0: exp(i pi q) sin(pi q) / (pi q).
struct DriftResponse {
    double z, half, root;  // |z|, |z| / 2, sqrt(2 / |z|)
    c64 e2q;               // exp(2 pi i q), the same for every integer shift of q (conjugated for z < 0)
    bool neg, narrow;      // z < 0; both ends of a bin inside can lie within 1 of 0

    __device__ DriftResponse(double r, double zz) {
        neg = zz < 0.0;
        z = fabs(zz);
        half = 0.5 * z;
        root = z > 0.0 ? sqrt(2.0 / z) : 0.0;
        narrow = z < 2.0;
        e2q = cis_pi(2.0 * r);
        if (neg) e2q.im = -e2q.im;
    }

    // A(q, z) sqrt(2 |z|) (z = 0: A(q, 0)).
    __device__ __forceinline__ c64 at(double q) const {
        if (z == 0.0) {
            if (q == rint(q)) return q == 0.0 ? c64{1.0, 0.0} : c64{0.0, 0.0};
            return cscale(cis_pi(q), sinpi(q) / (kPiD * q));
        }
        const double p = (neg ? -q : q) - half;
        const double Y = p * root, Zv = (p + z) * root;
        const c64 gy = fresnel_aux(fabs(Y)), gz = cmul(e2q, fresnel_aux(fabs(Zv)));
        const double sy = Y < 0.0 ? -1.0 : 1.0, sz = Zv < 0.0 ? 1.0 : -1.0;
        c64 a = {fma(sy, gy.re, sz * gz.re), fma(sy, gy.im, sz * gz.im)};
        const bool inside = Y < 0.0 && Zv >= 0.0;
        if (__any(inside)) {
            const c64 rot = cis_pi(-0.5 * Y * Y);
            if (inside) a = {a.re + (rot.re - rot.im), a.im + (rot.re + rot.im)};
            if (narrow) {
                const bool both = fabs(Y) < 1.0 && fabs(Zv) < 1.0;
                if (__any(both)) {
                    const c64 d = cmul(rot, csub(fresnel_small(Zv), fresnel_small(Y)));
                    if (both) a = d;
                }
            }
        }
        return neg ? c64{a.re, -a.im} : a;
    }
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Normalised spectrum value Xhat[k] = X[k] sqrt(ln2 / m(k)) (X itself when
// med is NULL), in FP64.
struct Spectrum {
    const float2 *X;
    const double *med;
    int W;
    int64_t nb, nblk;
    __device__ c64 at(int64_t k) const {
        const float2 x = X[k];
        const double f = med ? norm_scale(median_curve(med, nblk, W, nb, k)) : 1.0;
        return {double(x.x) * f, double(x.y) * f};
    }
};

// P(r, z) by one wave: Y = sum_{k in K(r)} Xhat[k] conj(A(r - k, z)) over the
// bins within h of r, normalised by sum_{k in K(r)} |A(r - k, z)|^2; Xhat is
// zero outside [0, nb).  The result is valid in every lane.
// (r, z) must be finite and below 2^50 in magnitude (NaN otherwise), so
// that the 2h or 2h + 1 offsets r - k are exact.
__device__ double wave_power(const Spectrum &sp, int h, double r, double z, int lane) {
    if (!(fabs(r) < 0x1p50) || !(fabs(z) < 0x1p50)) return NAN;
    const double klo = ceil(r - double(h));
    const int ntap = int(floor(r + double(h)) - klo) + 1;  // 2h or 2h + 1
    double nre = 0.0, nim = 0.0, den = 0.0;
    const DriftResponse resp(r, z);
    for (int t = lane; t < ntap; t += 64) {
        const double kk = klo + double(t);
        const c64 a = resp.at(r - kk);  // its constant factor leaves the power as it is
        den += cnorm2(a);
        const int64_t k = int64_t(kk);
        if (k >= 0 && k < sp.nb) {
            const c64 x = sp.at(k);
            nre += x.re * a.re + x.im * a.im;  // x conj(a)
            nim += x.im * a.re - x.re * a.im;
        }
    }
    nre = wave_sum(nre);
    nim = wave_sum(nim);
    den = wave_sum(den);
    return (nre * nre + nim * nim) / den;
}

// Point i (0..7) of a search level around (r, z): z-offset major, then
// r-offset, each in -1, 0, +1, the centre skipped.
__device__ __forceinline__ void level_point(int i, double r, double z, double sr, double sz, double &rr,
                                            double &zz) {
    const int g = i < 4 ? i : i + 1;
    const int b = g / 3 - 1, a = g % 3 - 1;
    rr = r + double(a) * sr;
    zz = z + double(b) * sz;
}

// The workgroup's harmonic sums S(r_i, z_i) = sum_{j=1}^{nh} P(j r_i, j z_i)
// for npts points (the level's neighbours, or the centre when npts is 1):
// waves take the (point, harmonic) pairs in turn, the per-pair powers meet in
// LDS (pw) and thread i sums point i's in the order j = 1 .. nh into S[i].
// On return S is visible to every thread.
__device__ void eval_points(const Spectrum &sp, int h, int nh, int npts, double r, double z, double sr, double sz,
                            double *pw, double *S) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    for (int pj = wave; pj < npts * nh; pj += nwaves) {
        const int i = pj / nh, j = pj - i * nh + 1;
        double rr = r, zz = z;
        if (npts > 1) level_point(i, r, z, sr, sz, rr, zz);
        const double p = wave_power(sp, h, double(j) * rr, double(j) * zz, lane);
        if (lane == 0) pw[pj] = p;
    }
    __syncthreads();
    if (int(threadIdx.x) < npts) {
        double s = 0.0;
        for (int j = 0; j < nh; ++j) s += pw[threadIdx.x * nh + j];
        S[threadIdx.x] = s;
    }
    __syncthreads();
}

// One workgroup per candidate (persistent grid): start at the fundamental
// r = k / (nh cpb), z = ((iz - izc) dz) / nh (cpb = 2 on a half-bin plane), then per level l = 1 .. levels move
// to the best of the 8 neighbours at steps (2^-l / nh, (dz 2^-l) / nh) when
// it is strictly larger than the centre (earlier points win ties); points
// whose top harmonic drifts beyond the bank (|nh z| > zmax) are skipped.
__global__ __launch_bounds__(RF_THREADS) void k_refine(Spectrum sp, int h, int izc, double dz, double zmax,
                                                       int cpb, int levels, const uint32_t *__restrict__ count,
                                                       uint32_t cap, fdas_cand *__restrict__ cands) {
    __shared__ double pw[RF_POINTS * RF_MAX_NH];
    __shared__ double S[RF_POINTS];
    const uint32_t n = min(*count, cap);
    for (uint32_t c = blockIdx.x; c < n; c += gridDim.x) {
        const int64_t k = cands[c].k;
        const int iz = cands[c].iz;
        const int nh = cands[c].nharm;
        if (nh < 1 || nh > RF_MAX_NH) continue;  // uniform over the workgroup
        double r = double(k) / (double(nh) * double(cpb));
        double z = (double(iz - izc) * dz) / double(nh);
        double best = 0.0;
        // level 0 evaluates the centre alone
        for (int l = 0; l <= levels; ++l) {
            const double sr = ldexp(1.0, -l) / double(nh);
            const double sz = (dz * ldexp(1.0, -l)) / double(nh);
            eval_points(sp, h, nh, l == 0 ? 1 : RF_POINTS, r, z, sr, sz, pw, S);
            if (l == 0) {
                best = S[0];
                continue;
            }
            double br = r, bz = z;
            for (int i = 0; i < RF_POINTS; ++i) {
                double rr, zz;
                level_point(i, r, z, sr, sz, rr, zz);
                if (fabs(double(nh) * zz) > zmax) continue;
                if (S[i] > best) {
                    best = S[i];
                    br = rr;
                    bz = zz;
                }
            }
            r = br;
            z = bz;
        }
        if (threadIdx.x == 0) {
            cands[c].r = r;
            cands[c].z = z;
            cands[c].power = float(best);
        }
    }
}

// Significance of the refined records' powers, one thread per record (kept
// out of k_refine, where its special functions would set the register budget
// of the whole search).
__global__ __launch_bounds__(256) void k_refine_sigma(const uint32_t *__restrict__ count, uint32_t cap,
                                                      fdas_cand *__restrict__ cands) {
    const uint32_t n = min(*count, cap);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int nh = cands[i].nharm;
        if (nh < 1 || nh > RF_MAX_NH) continue;
        cands[i].sigma = float(significance_d(double(cands[i].power), nh));
    }
}

// ------------------------------------------------ level by level
// The same search for a known, moderate number of records: one launch per
// level, a wave per (record, point, harmonic), so that records of 16 harmonics
// (784 evaluations of P at 6 levels) are spread over the GPU instead of
// holding one compute unit each.  The powers and the state a level starts
// from are kept per record, those of even and odd levels apart: a level's
// waves each work out the previous level's choice for themselves while it is
// being stored for the next.  Bit for bit the results of k_refine.
constexpr int RL_THREADS = 256;
constexpr int RL_PAIRS = RF_POINTS * RF_MAX_NH;

struct RefineState {
    double r, z, best;
};
struct RefineScratch {
    double *pw;          // [2][n][RL_PAIRS]
    RefineState *state;  // [2][n]
    uint32_t n;
};

// Where the search stands after `level` was evaluated (by a whole wave, the
// same in every lane).
__device__ RefineState after_level(const RefineScratch &sc, uint32_t rec, int level, int nh, double dz, double zmax,
                                   int lane) {
    RefineState st = sc.state[size_t(level & 1) * sc.n + rec];
    const double *__restrict__ pw = sc.pw + (size_t(level & 1) * sc.n + rec) * RL_PAIRS;
    double sum = 0.0;  // of point `lane`, in the order of the harmonics
    if (lane < (level == 0 ? 1 : RF_POINTS)) {
        double p[RF_MAX_NH];
#pragma unroll
        for (int j = 0; j < RF_MAX_NH; ++j) p[j] = j < nh ? pw[lane * nh + j] : 0.0;
#pragma unroll
        for (int j = 0; j < RF_MAX_NH; ++j)
            if (j < nh) sum += p[j];
    }
    if (level == 0) {
        st.best = __shfl(sum, 0);
        return st;
    }
    const double sr = ldexp(1.0, -level) / double(nh);
    const double sz = (dz * ldexp(1.0, -level)) / double(nh);
    const double r = st.r, z = st.z;
    for (int i = 0; i < RF_POINTS; ++i) {
        const double si = __shfl(sum, i);
        double rr, zz;
        level_point(i, r, z, sr, sz, rr, zz);
        if (fabs(double(nh) * zz) > zmax) continue;
        if (si > st.best) st = RefineState{rr, zz, si};
    }
    return st;
}

__global__ __launch_bounds__(RL_THREADS) void k_refine_level(Spectrum sp, int h, int izc, double dz, double zmax, int cpb,
                                                             int level, RefineScratch sc,
                                                             const fdas_cand *__restrict__ cands) {
    const int lane = threadIdx.x & 63;
    const int pair = int(blockIdx.y) * (RL_THREADS / 64) + int(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
    const uint32_t rec = blockIdx.x;
    const int nh = __builtin_amdgcn_readfirstlane(cands[rec].nharm);
    if (nh < 1 || nh > RF_MAX_NH || pair >= (level == 0 ? 1 : RF_POINTS) * nh) return;
    RefineState st;
    if (level == 0) {
        st.r = double(cands[rec].k) / (double(nh) * double(cpb));
        st.z = (double(cands[rec].iz - izc) * dz) / double(nh);
        st.best = 0.0;
    } else {
        st = after_level(sc, rec, level - 1, nh, dz, zmax, lane);
    }
    if (pair == 0 && lane == 0) sc.state[size_t(level & 1) * sc.n + rec] = st;
    const int i = pair / nh, j = pair - i * nh + 1;
    double rr = st.r, zz = st.z;
    if (level > 0)
        level_point(i, st.r, st.z, ldexp(1.0, -level) / double(nh), (dz * ldexp(1.0, -level)) / double(nh), rr, zz);
    const double p = wave_power(sp, h, double(j) * rr, double(j) * zz, lane);
    if (lane == 0) sc.pw[(size_t(level & 1) * sc.n + rec) * RL_PAIRS + pair] = p;
}

// The records' final points and their significance, a wave per record.
__global__ __launch_bounds__(64) void k_refine_result(double dz, double zmax, int levels, RefineScratch sc,
                                                      fdas_cand *__restrict__ cands) {
    const uint32_t rec = blockIdx.x;
    const int nh = cands[rec].nharm;
    if (nh < 1 || nh > RF_MAX_NH) return;
    const RefineState st = after_level(sc, rec, levels, nh, dz, zmax, threadIdx.x);
    if (threadIdx.x == 0) {
        const float power = float(st.best);
        cands[rec].r = st.r;
        cands[rec].z = st.z;
        cands[rec].power = power;
        cands[rec].sigma = float(significance_d(double(power), nh));
    }
}

// S(r_i, z_i) for listed points, one workgroup per point (persistent grid).
__global__ __launch_bounds__(RF_POINT_THREADS) void k_interp_points(Spectrum sp, int h, const double *__restrict__ r,
                                                              const double *__restrict__ z,
                                                              const int32_t *__restrict__ nh, int64_t n,
                                                              double *__restrict__ out) {
    __shared__ double pw[RF_MAX_NH];
    __shared__ double S[1];
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int m = nh[i];
        if (m < 1 || m > RF_MAX_NH) {
            if (threadIdx.x == 0) out[i] = NAN;
            continue;
        }
        eval_points(sp, h, m, 1, r[i], z[i], 0.0, 0.0, pw, S);
        if (threadIdx.x == 0) out[i] = S[0];
    }
}

Spectrum make_spectrum(const float2 *X, const double *med, int W, int64_t nb) {
    Spectrum sp;
    sp.X = X;
    sp.med = med;
    sp.W = W;
    sp.nb = nb;
    sp.nblk = (nb + W - 1) / W;
    return sp;
}

}  // namespace

hipError_t launch_refine(const float2 *X, const double *med, int W, int64_t nb, int h, int izc, double dz,
                         double zmax, int cpb, int levels, const uint32_t *count, uint32_t cap, fdas_cand *cands,
                         int workgroups, hipStream_t st) {
    if (cap == 0 || levels <= 0) return hipSuccess;
    if (levels > 30 || workgroups <= 0 || nb <= 0 || W <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_refine, dim3(unsigned(workgroups)), dim3(RF_THREADS), 0, st,
                       make_spectrum(X, med, W, nb), h, izc, dz, zmax, cpb, levels, count, cap, cands);
    hipLaunchKernelGGL(k_refine_sigma, dim3(unsigned(workgroups)), dim3(256), 0, st, count, cap, cands);
    return hipGetLastError();
}

size_t refine_level_scratch_bytes(int64_t n) {
    return size_t(2 * n) * (RL_PAIRS * sizeof(double) + sizeof(RefineState));
}

hipError_t launch_refine_levels(const float2 *X, const double *med, int W, int64_t nb, int h, int izc, double dz,
                                double zmax, int cpb, int levels, int64_t n, fdas_cand *cands, void *scratch_dev,
                                hipStream_t st) {
    if (n <= 0 || n > kRefineLevelsMost || levels < 1 || levels > 30 || nb <= 0 || W <= 0) return hipErrorInvalidValue;
    RefineScratch sc;
    sc.pw = static_cast<double *>(scratch_dev);
    sc.state = reinterpret_cast<RefineState *>(sc.pw + size_t(2 * n) * RL_PAIRS);
    sc.n = uint32_t(n);
    for (int level = 0; level <= levels; ++level) {
        const int pairs = level == 0 ? RF_MAX_NH : RL_PAIRS;
        hipLaunchKernelGGL(k_refine_level, dim3(unsigned(n), unsigned(pairs / (RL_THREADS / 64))), dim3(RL_THREADS), 0,
                           st, make_spectrum(X, med, W, nb), h, izc, dz, zmax, cpb, level, sc, cands);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_refine_result, dim3(unsigned(n)), dim3(64), 0, st, dz, zmax, levels, sc, cands);
    return hipGetLastError();
}

// Records, count and level scratch of fdas_refine_noalloc: a file-scope device
// array, one copy per GPU, held until the process ends.  Host code never hands the
// array's name to a kernel or a copy (on the host it is only a stand-in for
// the symbol); it uses the device address hipGetSymbolAddress returns for
// the current device, looked up once per device and kept.
constexpr size_t kRefineScratchBytes = size_t(FDAS_REFINE_NOALLOC_MAX) * sizeof(fdas_cand) + 256 +
                                       size_t(2 * kRefineLevelsMost) * (RL_PAIRS * sizeof(double) + sizeof(RefineState));
static __device__ __align__(256) unsigned char scratch[kRefineScratchBytes];

hipError_t refine_noalloc_scratch(void **out, size_t *bytes) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *out = addr[dev];
    *bytes = kRefineScratchBytes;
    return hipSuccess;
}

hipError_t launch_interp_points(const float2 *X, const double *med, int W, int64_t nb, int h, const double *r,
                                const double *z, const int32_t *nh, int64_t n, double *out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (nb <= 0 || W <= 0) return hipErrorInvalidValue;
    const int64_t grid = n < 4096 ? n : 4096;
    hipLaunchKernelGGL(k_interp_points, dim3(unsigned(grid)), dim3(RF_POINT_THREADS), 0, st,
                       make_spectrum(X, med, W, nb), h, r, z, nh, n, out);
    return hipGetLastError();
}

}  // namespace fdas
