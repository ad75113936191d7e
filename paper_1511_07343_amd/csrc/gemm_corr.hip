// Precision variant of the correlation: Eq. (1) of Sec. 2 evaluated directly,
// as one real matrix product on the MFMA units with BF16 or FP16 operands and
// FP32 accumulation, instead of the overlap-save FFT path.
//
// Y_z[k] = sum_{q=-h..h} Xhat[k - q] T_z[q].  At integer offsets the response
// of Sec. 2 is even in q and A(q, -z) = conj A(-q, z), so with T_z = C + i D
// (real and imaginary parts of the taps) T_-z = C - i D, and the four real
// products of a pair of templates +-z,
//   Ur = Re Xhat * C,  Ui = Im Xhat * C,  Vr = Re Xhat * D,  Vi = Im Xhat * D,
// give both: Y_z = (Ur - Vi) + i (Ui + Vr), Y_-z = (Ur + Vi) + i (Ui - Vr).
// That is half the multiplications of one product per template.  With
// q' = q + h, a product is A B, A[k][q'] = Xhat[k - q' + h] (its real or
// imaginary part) and B the taps.  A is a Toeplitz matrix: row k + 1 is row k
// shifted by one value, so a block of rows needs only a window of the
// spectrum.  The powers |Y|^2 and their screening codes go to the same plane
// layout the FFT path writes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <vector>

#include "device_common.hpp"
#include "kernels.hpp"

namespace fdas {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// v_mfma_f32_32x32x16_{bf16,f16}: lane l holds A[l % 32][8 (l / 32) + s] and
// B[8 (l / 32) + s][l % 32] (s < 8) and receives
// D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32] (r < 16).
template <bool BF16>
__device__ __forceinline__ f32x16 mfma(uint4 a, uint4 b, f32x16 c) {
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                      0, 0);
}

// 16-bit encodings, round to nearest even (the same conversions on host and
// device).
template <bool BF16>
__host__ __device__ inline uint16_t to_half_bits(float x) {
    if constexpr (BF16) return __builtin_bit_cast(uint16_t, static_cast<__bf16>(x));
    else return __builtin_bit_cast(uint16_t, static_cast<_Float16>(x));
}

constexpr int GM_WAVES = 4;
constexpr int GM_RT = 4;                         // row tiles of 32 bins per wave
constexpr int GM_ROWS = GM_WAVES * GM_RT * 32;   // bins per row block
constexpr int GM_PAIRS = 16;                     // template pairs per slice: columns C, then D
constexpr int GM_WIN = 8;                        // A fragments of each part kept per wave
constexpr int GM_FRAG = 64;                      // 16-byte fragments per MFMA operand (one per lane)
constexpr int GM_WORDS(int nk) { return GM_ROWS + 16 * nk; }  // window values (a multiple of 8)
// Bytes from one copy of the window to the next: 32 more than a multiple of
// 256, so that the 16 lanes of a fragment read that take eight copies, two
// neighbouring pieces each, cover 256 consecutive bytes' worth of banks.
constexpr int GM_STRIDE(int nk) { return (2 * GM_WORDS(nk) - 32 + 255) / 256 * 256 + 32; }

static_assert(GM_WORDS(GM_MAX_KSTEPS) / 8 <= 64 * GM_WAVES, "8 window values per thread");

// FP16 taps are scaled by 16 (exactly), which keeps the tails of the templates
// away from its subnormal range, and their powers back by 1/256.  BF16 has the
// range of FP32 and needs neither.
constexpr double gm_tap_scale(bool bf16) { return bf16 ? 1.0 : 16.0; }

// Word k = (Re, Im) of Xhat[k] as two 16-bit floats, Re in the low half.
template <bool BF16>
__global__ __launch_bounds__(256) void k_lowp_spectrum(const float2 *__restrict__ X, const double *__restrict__ med,
                                                       int W, int64_t nb, uint32_t *__restrict__ out,
                                                       uint32_t *__restrict__ counters) {
    if (blockIdx.x == 0 && threadIdx.x < 6) counters[threadIdx.x] = 0u;
    const int64_t g = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (g >= nb) return;
    float2 x = X[g];
    if (med) {
        const int64_t nblk = (nb + W - 1) / W;
        const double mk = median_curve(med, nblk, W, nb, g);
        const float sc = float(norm_scale(mk));
        x = make_float2(x.x * sc, x.y * sc);
    }
    out[g] = uint32_t(to_half_bits<BF16>(x.x)) | (uint32_t(to_half_bits<BF16>(x.y)) << 16);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_nt(float *p, const float (&v)[4]) {
    __builtin_nontemporal_store(f32x4{v[0], v[1], v[2], v[3]}, reinterpret_cast<f32x4 *>(p));
}

// Codes of 128 bins of one template, spread over the four lanes l % 16 + 16 j:
// lane j' = 2 ((l / 16) % 2) + l / 32 holds the two codes of bins
// 32 rt + 8 g + 4 j' .. + 3 of tile rt in the low (g = 0) and the high (g = 2)
// half of w[rt].  On return, the 16 codes of tile j' in bin order.
__device__ __forceinline__ uint4 gather_codes(const uint32_t (&w)[GM_RT]) {
    static_assert(GM_RT == 4, "a tile per lane");
    const auto a = __builtin_amdgcn_permlane32_swap(w[0], w[1], false, false);  // a[e]: from lanes l / 32 = e,
    const auto b = __builtin_amdgcn_permlane32_swap(w[2], w[3], false, false);  // tile l / 32 (b: + 2)
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);  // c[hi]: from (l / 16) % 2 = hi, e = 0
    const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);  // ... e = 1
    constexpr uint32_t lo = 0x05040100u, hi = 0x07060302u;  // the low (high) halves of two words
    return make_uint4(__builtin_amdgcn_perm(d[0], c[0], lo), __builtin_amdgcn_perm(d[1], c[1], lo),
                      __builtin_amdgcn_perm(d[0], c[0], hi), __builtin_amdgcn_perm(d[1], c[1], hi));
}

// One workgroup: the B fragments of one slice of 16 template pairs (all K)
// staged in LDS, then row blocks of GM_ROWS bins, each through a spectrum
// window in LDS.  Wave w owns rows [128 w, 128 w + 128) of a block (4 row
// tiles) times 32 columns (C and D of the pairs), once for the real and once
// for the imaginary part of the spectrum: 8 accumulators, 8 products per K
// step of 16 for 3 fragment reads.
//
// The A fragment of (row tile rt, K step ks) holds the 8 window values from
// u = (GM_ROWS - 1 - row) + 16 ks + 8 (l / 32) on, which depend on ks - 2 rt
// only: F(d) with d = ks - 2 rt.  A wave keeps F(ks - 6) .. F(ks + 1) of each
// part in registers and loads one new fragment of each per K step.  The
// window is stored in eight copies shifted by one value, so that every
// lane's fragment is a 16-byte aligned LDS read (copy (7 - l) mod 8).
//
// The next block's window is loaded into registers before this block's
// powers are stored, so that the stores drain while the next block runs
// (vector-memory counters count loads and stores together).
template <bool BF16>
__global__ __launch_bounds__(64 * GM_WAVES, 2) void k_corr_gemm(
    const uint32_t *__restrict__ xl, int64_t nb, int h, int nk, const uint4 *__restrict__ bfrag, int nz, int nsl,
    int64_t nrb, int64_t per, float *__restrict__ plane, uint8_t *__restrict__ codes,
    float code_inv) {
    extern __shared__ uint4 gm_lds[];
    uint4 *__restrict__ bl = gm_lds;  // nk GM_FRAG fragments
    // then 8 copies of the real parts' window, 8 of the imaginary parts'
    char *__restrict__ win = reinterpret_cast<char *>(gm_lds + nk * GM_FRAG);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int uw = GM_WORDS(nk), ust = GM_STRIDE(nk);
    const int sig = (7 - lane) & 7;
    // byte of F(0) of the real parts in copy sig; F(d) is 32 d bytes further
    const char *__restrict__ fr = win + sig * ust + 2 * (GM_ROWS - 1 - 128 * wave - (lane & 31) + 8 * (lane >> 5) - sig);
    const char *__restrict__ fi = fr + 8 * ust;
    auto frag = [](const char *p, int d) { return *reinterpret_cast<const uint4 *>(p + 32 * d); };

    // this workgroup's items: (slice, row block) pairs [item0, item1), slice-major
    const int64_t total = int64_t(nsl) * nrb;
    const int64_t item0 = int64_t(blockIdx.x) * per;
    const int64_t item1 = min(total, item0 + per);
    if (item0 >= item1) return;
    // window values W[u] = xl[P0 - u] (zero outside the spectrum), thread t
    // holding u = 8 t .. 8 t + 14, of which copy s takes W[8 t + s] .. + 7
    constexpr int NW = 15;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(xl), short(0), int(4 * nb), 0x00020000);
    uint32_t wreg[NW];
    const bool fills = 8 * t < uw;
    auto load_window = [&](int64_t item) {
        const int sl = int(item / nrb);
        const int p0 = int(item - int64_t(sl) * nrb) * GM_ROWS + GM_ROWS - 1 + h - 8 * t;
        if (fills) {  // bytes outside the spectrum, before (negative, a large unsigned offset) or past it, read 0
#pragma unroll
            for (int i = 0; i < NW; ++i) wreg[i] = __builtin_amdgcn_raw_buffer_load_b32(rx, 4 * (p0 - i), 0, 0);
        }
    };
    load_window(item0);
    const int pairs = (nz + 1) / 2;
    int cur_slice = -1;
    for (int64_t item = item0; item < item1; ++item) {
        const int sl = int(item / nrb);
        const int64_t k0 = (item - int64_t(sl) * nrb) * GM_ROWS;
        __syncthreads();  // the previous item's LDS reads are done
        if (sl != cur_slice) {
            const uint4 *__restrict__ src = bfrag + int64_t(sl) * nk * GM_FRAG;
            for (int i = t; i < nk * GM_FRAG; i += 64 * GM_WAVES) bl[i] = src[i];
            cur_slice = sl;
        }
        if (fills) {
#pragma unroll
            for (int part = 0; part < 2; ++part) {
                uint32_t pr[NW - 1];  // (W[i], W[i + 1]) of this part
#pragma unroll
                for (int i = 0; i < NW - 1; ++i)
                    pr[i] = __builtin_amdgcn_perm(wreg[i + 1], wreg[i], part ? 0x07060302u : 0x05040100u);
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    *reinterpret_cast<uint4 *>(win + (8 * part + c) * ust + 16 * t) =
                        make_uint4(pr[c], pr[c + 2], pr[c + 4], pr[c + 6]);
            }
        }
        __syncthreads();

        f32x16 acc[GM_RT][2];
#pragma unroll
        for (int rt = 0; rt < GM_RT; ++rt)
#pragma unroll
            for (int part = 0; part < 2; ++part)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[rt][part][r] = 0.f;
        uint4 Fr[GM_WIN], Fi[GM_WIN];
#pragma unroll
        for (int d = 0; d <= 2 * (GM_RT - 1); ++d) {  // F(0), F(-1) .. F(-6)
            Fr[(GM_WIN - d) % GM_WIN] = frag(fr, -d);
            Fi[(GM_WIN - d) % GM_WIN] = frag(fi, -d);
        }
        uint4 b = bl[lane];
        for (int kb = 0; kb < nk; kb += GM_WIN) {
#pragma unroll
            for (int j = 0; j < GM_WIN; ++j) {
                const int ks = kb + j;
                if (ks < nk) {
                    // prefetch step ks + 1 (F(ks + 1) replaces F(ks - 7), no longer used)
                    uint4 bn = b;
                    if (ks + 1 < nk) {
                        Fr[(j + 1) % GM_WIN] = frag(fr, ks + 1);
                        Fi[(j + 1) % GM_WIN] = frag(fi, ks + 1);
                        bn = bl[(ks + 1) * GM_FRAG + lane];
                    }
#pragma unroll
                    for (int rt = 0; rt < GM_RT; ++rt) {
                        acc[rt][0] = mfma<BF16>(Fr[(j - 2 * rt + GM_WIN) % GM_WIN], b, acc[rt][0]);
                        acc[rt][1] = mfma<BF16>(Fi[(j - 2 * rt + GM_WIN) % GM_WIN], b, acc[rt][1]);
                    }
                    b = bn;
                }
            }
        }
        if (item + 1 < item1) load_window(item + 1);

        // Powers.  Lanes with l % 32 < 16 hold U of pair l % 16, the others V:
        // exchanging registers 4 g + i and 4 (g + 1) + i between the odd and
        // the even rows of 16 lanes leaves both of U and V of 4 consecutive
        // bins in every lane (of the tile's group g or g + 1 of 8 bins).
        const int pr = sl * GM_PAIRS + (lane & 15);
        if (pr < pairs) {
            const int mirror = nz - 1 - pr;
            const int64_t kw = k0 + 128 * wave;
            float *__restrict__ prow = plane + int64_t(pr) * nb + kw, *__restrict__ mrow = plane + int64_t(mirror) * nb + kw;
            uint32_t pc[GM_RT], mc[GM_RT];  // codes of each tile: group g = 0 low, 2 high
#pragma unroll
            for (int rt = 0; rt < GM_RT; ++rt) {
#pragma unroll
                for (int g = 0; g < 4; g += 2) {
                    float pz[4], pm[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const auto r = __builtin_amdgcn_permlane16_swap(
                            __float_as_uint(acc[rt][0][4 * g + i]), __float_as_uint(acc[rt][0][4 * (g + 1) + i]), false, false);
                        const auto m = __builtin_amdgcn_permlane16_swap(
                            __float_as_uint(acc[rt][1][4 * g + i]), __float_as_uint(acc[rt][1][4 * (g + 1) + i]), false, false);
                        const float ur = __uint_as_float(r[0]), vr = __uint_as_float(r[1]);
                        const float ui = __uint_as_float(m[0]), vi = __uint_as_float(m[1]);
                        const float ar = ur - vi, ai = ui + vr, br = ur + vi, bi = ui - vr;
                        pz[i] = fmaf(ar, ar, ai * ai);
                        pm[i] = fmaf(br, br, bi * bi);
                        if constexpr (!BF16) {
                            constexpr float scale = float(1.0 / (gm_tap_scale(false) * gm_tap_scale(false)));
                            pz[i] *= scale;
                            pm[i] *= scale;
                        }
                    }
                    const int k = 32 * rt + 8 * (g + ((lane >> 4) & 1)) + 4 * (lane >> 5);
                    store_nt(prow + k, pz);
                    if (mirror != pr) store_nt(mrow + k, pm);
                    const uint32_t cp = block_codes4(make_float4(pz[0], pz[1], pz[2], pz[3]), code_inv);
                    const uint32_t cm = block_codes4(make_float4(pm[0], pm[1], pm[2], pm[3]), code_inv);
                    pc[rt] = g == 0 ? cp : pc[rt] | (cp << 16);
                    mc[rt] = g == 0 ? cm : mc[rt] | (cm << 16);
                }
            }
            const int tile = 2 * ((lane >> 4) & 1) + (lane >> 5);  // the tile whose codes this lane stores
            uint8_t *__restrict__ code0 = codes + kw / 2 + 16 * tile;
            *reinterpret_cast<uint4 *>(code0 + int64_t(pr) * (nb / 2)) = gather_codes(pc);
            if (mirror != pr) *reinterpret_cast<uint4 *>(code0 + int64_t(mirror) * (nb / 2)) = gather_codes(mc);
        }
    }
}

}  // namespace

int gemm_ksteps(int h) { return (2 * h + 1 + 15) / 16; }

static size_t gemm_lds_bytes(int nk) { return size_t(nk) * GM_FRAG * 16 + 16 * size_t(GM_STRIDE(nk)); }

static int gemm_slices(int nz) { return ((nz + 1) / 2 + GM_PAIRS - 1) / GM_PAIRS; }

size_t gemm_bank_bytes(int nz, int h) { return size_t(gemm_slices(nz)) * size_t(gemm_ksteps(h)) * GM_FRAG * 16; }

// The taps of templates 0 .. (nz - 1) / 2; the others are their conjugates.
void build_gemm_bank(const double *taps, int nz, int h, bool bf16, void *out) {
    const int ntap = 2 * h + 1, nk = gemm_ksteps(h), nsl = gemm_slices(nz), pairs = (nz + 1) / 2;
    uint16_t *o = static_cast<uint16_t *>(out);
    size_t idx = 0;
    for (int sl = 0; sl < nsl; ++sl)
        for (int ks = 0; ks < nk; ++ks)
            for (int l = 0; l < 64; ++l)
                for (int s = 0; s < 8; ++s, ++idx) {
                    const int qp = 16 * ks + 8 * (l / 32) + s;
                    const int col = l % 32, z = sl * GM_PAIRS + col % GM_PAIRS, part = col / GM_PAIRS;
                    const double v = qp < ntap && z < pairs ? taps[2 * (size_t(z) * ntap + qp) + part] : 0.0;
                    const float f = float(v * gm_tap_scale(bf16));
                    o[idx] = bf16 ? to_half_bits<true>(f) : to_half_bits<false>(f);
                }
}

hipError_t launch_lowp_spectrum(const float2 *X, const double *med, int W, int64_t nb, bool bf16, uint32_t *out,
                                uint32_t *counters, hipStream_t st) {
    if (nb <= 0) return hipSuccess;
    const dim3 grid(unsigned((nb + 255) / 256));
    if (bf16) hipLaunchKernelGGL(k_lowp_spectrum<true>, grid, dim3(256), 0, st, X, med, W, nb, out, counters);
    else hipLaunchKernelGGL(k_lowp_spectrum<false>, grid, dim3(256), 0, st, X, med, W, nb, out, counters);
    return hipGetLastError();
}

hipError_t launch_corr_gemm(const uint32_t *xl, int64_t nb, int h, const void *bank, int nz, bool bf16,
                            int workgroups, float *plane, uint8_t *codes, float code_inv, hipStream_t st) {
    const int nk = gemm_ksteps(h);
    if (nk > GM_MAX_KSTEPS || nb % GM_ROWS != 0 || nb > (int64_t(1) << 28) || workgroups <= 0) return hipErrorInvalidValue;
    const int nsl = gemm_slices(nz);
    const int64_t nrb = (nb + GM_ROWS - 1) / GM_ROWS;
    const size_t lds = gemm_lds_bytes(nk);
    // workgroups per CU that fit beside each other (the LDS decides)
    int per_cu = 0;
    hipError_t e = bf16 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_corr_gemm<true>, 64 * GM_WAVES, lds)
                        : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_corr_gemm<false>, 64 * GM_WAVES, lds);
    if (e != hipSuccess) return e;
    workgroups *= std::max(per_cu, 1);
    const int64_t per = (int64_t(nsl) * nrb + workgroups - 1) / workgroups;
    const int64_t grid = (int64_t(nsl) * nrb + per - 1) / per;
    const uint4 *bf = static_cast<const uint4 *>(bank);
    if (bf16)
        hipLaunchKernelGGL(k_corr_gemm<true>, dim3(unsigned(grid)), dim3(64 * GM_WAVES), lds, st, xl, nb, h, nk, bf, nz,
                           nsl, nrb, per, plane, codes, code_inv);
    else
        hipLaunchKernelGGL(k_corr_gemm<false>, dim3(unsigned(grid)), dim3(64 * GM_WAVES), lds, st, xl, nb, h, nk, bf,
                           nz, nsl, nrb, per, plane, codes, code_inv);
    return hipGetLastError();
}

}  // namespace fdas
