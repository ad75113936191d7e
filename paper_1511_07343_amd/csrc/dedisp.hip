// De-dispersion (the step before the search, Sec. 1: one time series per
// dispersion-measure trial): the channels of a channel-major 8-bit
// filterbank shifted by their per-DM sample delays and added, in exact
// integer arithmetic on the matrix cores.
#include "delays.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <cmath>

namespace fdas {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // rows start at any float

constexpr int kDdXcds = 8;

// The work items of one launch: workgroup i takes item
// first + (i mod 8) per + i div 8 if that lies below end, so that neighbouring
// items share an XCD's L2.
struct Items {
    int64_t first, end, per;
    __device__ __forceinline__ int64_t mine() const {
        return first + int64_t(blockIdx.x % kDdXcds) * per + blockIdx.x / kDdXcds;
    }
};

// launch(grid, items) for all of `total` work items, a workgroup of `threads`
// threads each, in as few launches as the runtime takes (a grid has less than
// 2^32 threads).
template <class Launch>
hipError_t launch_items(int64_t total, int threads, Launch launch) {
    const int64_t most = int64_t(0xffffffffu) / threads / kDdXcds * kDdXcds;
    for (int64_t first = 0; first < total; first += most) {
        const int64_t n = std::min(most, total - first), per = (n + kDdXcds - 1) / kDdXcds;
        launch(unsigned(per * kDdXcds), Items{first, first + n, per});
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

constexpr int kFlip = int(0x80808080u);  // b -> b - 128 as signed bytes

// 16 bytes, all 0 but a 1 at byte `at` (none outside 0 .. 15).
__device__ __forceinline__ i32x4 one_at(int at) {
    const int one = 1 << (8 * (at & 3));
    i32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (at >> 2) == i ? one : 0;
    return v;
}

// The sums on the matrix cores: one v_mfma_i32_16x16x64_i8 with A the 16 x 64
// matrix of four identities side by side adds 4 channels of 256 output
// samples: D[i][n] += sum_q B[16 q + i][n], lane n + 16 q of B holding the 16
// bytes of sample block n of channel q.  The samples' top bits are flipped
// (b - 128 as a signed byte) and 128 per channel added back at the end.

// A lane's four sums of a tile, samples t .. t + 3; those before `first` belong
// to another span.
__device__ __forceinline__ void store_sums(float *__restrict__ o, int64_t t, int64_t first, i32x4 sum) {
    const f32x4u v = {float(sum[0]), float(sum[1]), float(sum[2]), float(sum[3])};
    if (t >= first) {
        __builtin_nontemporal_store(v, reinterpret_cast<f32x4u *>(o + t));
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (t + r >= first) o[t + r] = v[r];
    }
}

// Start of a span: the last one of a series ends at nout (its first samples
// are those of the span before it, which stores them), so that every sample
// it adds up lies below nout + its delay.
__device__ __forceinline__ int64_t span_start(int64_t first, int span, int64_t nout) {
    return min(first, nout - span);
}

// ---------------------------------------------------------- through LDS
// A workgroup adds one span of 1280 samples for DL_GROUP consecutive DM
// trials, DL_DMS per wave.  In stages of DL_CH channels, each channel's bytes
// that any of the trials needs (the span and the spread of their delays,
// `row` bytes) are staged in LDS once, two stages in turn, and read from
// there by every trial.  LDS reads of 16 bytes run at full rate only when
// aligned, so a trial reads the aligned pieces that hold its samples and the
// matrix A does the byte shift: for samples that start at byte s of a piece,
// row i of A has its one at byte i + s of two pieces, and a block of 16
// samples takes two products, one with each.  A lane's blocks follow one
// another (block i of lane n is 5 n + i), so that the second piece of a block
// is the first of the next: 6 reads for 5 blocks of 4 channels, where blocks
// side by side in the lanes take 2 for each.  Five, because lanes 80 bytes
// apart fall on different banks.  64 channels to 256 trials of 2^23 samples in
// 4.99 ms (1.4e11 bytes added, 28 TB/s; LDS busy 58 % of the time, vector ALU
// 53 %, matrix cores 37 %: four waves a SIMD wait for one another's stages),
// against 5.39 ms with two reads a block, 7.3 ms with unaligned LDS reads and
// byte alignments in registers, 12.0 ms for the direct form and 14.2 ms for
// sums of 16-bit fields on the vector units.  Three blocks a lane take 6.0 ms,
// seven 5.8 (registers), both trials' reads together 5.7.
constexpr int DL_WAVES = 8;
constexpr int DL_DMS = 2;
constexpr int DL_GROUP = DL_WAVES * DL_DMS;
constexpr int DL_CH = 16;
constexpr int DL_TILES = 5;
constexpr int DL_SPAN = 256 * DL_TILES;
constexpr int DL_MAX_ROW = 2304;
constexpr int DL_LOADS = (DL_MAX_ROW + 511) / 512;  // 16-byte pieces per thread and stage

static_assert(DL_CH * 32 == DL_WAVES * 64, "32 threads stage a channel");
static_assert(DL_DMS + 1 <= 4, "a wave evaluates its trials' and the smallest delays in one go");

__global__ __launch_bounds__(64 * DL_WAVES, 4) void k_dedisperse_lds(const uint8_t *__restrict__ fil, int nchan,
                                                                  int64_t nsamp, Dispersion disp, int ndm, int64_t nout,
                                                                  int row, Items items, float *__restrict__ out) {
    extern __shared__ __align__(16) uint8_t stage[];  // 2 x DL_CH rows of `row` bytes
    const int64_t u = items.mine();
    if (u >= items.end) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4;
    const int ngrp = (ndm + DL_GROUP - 1) / DL_GROUP;
    const int64_t span = u / ngrp;
    const int dm0 = int(u - span * ngrp) * DL_GROUP, dm1 = min(ndm, dm0 + DL_GROUP);
    const int64_t first = span * DL_SPAN, t0 = span_start(first, DL_SPAN, nout);
    const int64_t fil_bytes = int64_t(nchan) * nsamp;
    // lanes 16 k ..: trial k of this wave (k < DL_DMS), then the group's smallest DM
    double kmin = disp.kdm[dm0];
    for (int i = dm0 + 1; i < dm1; ++i) kmin = fmin(kmin, disp.kdm[i]);
    const int mine = dm0 + wave * DL_DMS;
    const double kdm = q < DL_DMS ? disp.kdm[min(mine + q, dm1 - 1)] : kmin;
    const int my_ch = 2 * wave + (lane >> 5);  // the channel this thread stages

    i32x4 piece[DL_LOADS];
    int at = 0;  // lane 16 k + c: trial k's first byte in the row of channel c
    // The stage of channels c0 ..: this thread's pieces, and the offsets.
    auto fetch = [&](int c0) {
        const int c = min(c0 + (lane & 15), nchan - 1);
        const int d = delay_fast(disp, kdm, c);
        const int dmin = __shfl(d, 16 * DL_DMS + (lane & 15));
        const int rem = int((int64_t(c) * nsamp + t0 + dmin) & 3);
        at = (lane & 15) * row + rem + (d - dmin);
        const int64_t src = (int64_t(min(c0 + my_ch, nchan - 1)) * nsamp + t0 + __shfl(d, 16 * DL_DMS + my_ch)) & ~int64_t(3);
#pragma unroll
        for (int k = 0; k < DL_LOADS; ++k) {
            const int off = 16 * (lane & 31) + 512 * k;
            const int64_t a = src + off;
            piece[k] = i32x4{0, 0, 0, 0};
            if (off < row && c0 + my_ch < nchan) {
                if (a + 16 <= fil_bytes) {
                    piece[k] = *reinterpret_cast<const i32x4u *>(fil + a) ^ kFlip;
                } else {  // the last bytes of the filterbank
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        uint32_t w = 0;
                        for (int64_t i = a + 4 * j; i < min(fil_bytes, a + 4 * j + 4); ++i)
                            w |= uint32_t(fil[i]) << (8 * int(i - a - 4 * j));
                        piece[k][j] = int(w) ^ kFlip;
                    }
                }
            }
        }
    };
    auto put = [&](uint8_t *buf) {
#pragma unroll
        for (int k = 0; k < DL_LOADS; ++k) {
            const int off = 16 * (lane & 31) + 512 * k;
            if (off < row) *reinterpret_cast<i32x4 *>(buf + my_ch * row + off) = piece[k];
        }
    };

    i32x4 acc[DL_DMS][DL_TILES];
#pragma unroll
    for (int k = 0; k < DL_DMS; ++k)
#pragma unroll
        for (int i = 0; i < DL_TILES; ++i) acc[k][i] = i32x4{0, 0, 0, 0};
    const int buf_bytes = DL_CH * row;
    fetch(0);
    put(stage);
    __syncthreads();
    int cur = 0;
    for (int c0 = 0; c0 < nchan; c0 += DL_CH, cur ^= 1) {
        const int now = at;
        if (c0 + DL_CH < nchan) fetch(c0 + DL_CH);
        const uint8_t *__restrict__ buf = stage + cur * buf_bytes + 16 * DL_TILES * (lane & 15);
        // four channels at a time; the rows past the last channel are zero
#pragma unroll 1
        for (int g = 0; g < min(DL_CH, nchan - c0); g += 4) {
#pragma unroll
            for (int k = 0; k < DL_DMS; ++k) {
                const int o = __shfl(now, 16 * k + g + q);
                const uint8_t *__restrict__ p = buf + (o & ~15);
                i32x4 w[DL_TILES + 1];
#pragma unroll
                for (int i = 0; i <= DL_TILES; ++i) w[i] = *reinterpret_cast<const i32x4 *>(p + 16 * i);
                const int x = (lane & 15) + (o & 15);
                const i32x4 lo = one_at(x), hi = one_at(x - 16);
#pragma unroll
                for (int i = 0; i < DL_TILES; ++i)
                    acc[k][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(lo, w[i], acc[k][i], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < DL_TILES; ++i)
                    acc[k][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(hi, w[i + 1], acc[k][i], 0, 0, 0);
            }
        }
        // the other buffer was last read before the previous barrier
        if (c0 + DL_CH < nchan) put(stage + (cur ^ 1) * buf_bytes);
        __syncthreads();
    }
    // Through LDS, a region of the stage for each wave, so that a store covers
    // 256 consecutive samples (a lane's own blocks are 64 bytes each, 320
    // bytes apart: half lines of memory).
    static_assert(4 * DL_WAVES * DL_SPAN <= 2 * DL_CH * (DL_SPAN + 16), "the sums fit the smallest stage");
    i32x4 *const mem = reinterpret_cast<i32x4 *>(stage) + wave * (DL_SPAN / 4);
#pragma unroll
    for (int k = 0; k < DL_DMS; ++k) {
        if (mine + k >= dm1) break;
        float *__restrict__ o = out + int64_t(mine + k) * nout;
#pragma unroll
        for (int i = 0; i < DL_TILES; ++i) mem[4 * (DL_TILES * (lane & 15) + i) + q] = acc[k][i] + 128 * nchan;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int i = 0; i < DL_TILES; ++i) store_sums(o, t0 + 256 * i + 4 * lane, first, mem[64 * i + lane]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// ------------------------------------------------------------- directly
// One span of 256 TILES samples of one DM trial, the 16-byte blocks loaded
// from the filterbank at their byte addresses (through the L1, whose
// unaligned 16-byte loads bound it).  A workgroup's waves take one trial each,
// or (SPLIT) a quarter of the channels of one trial each, added up through
// LDS.
constexpr int DD_WAVES = 4;

// A wave's sums over channels [c0, c1).
template <int TILES>
struct ChannelSums {
    const uint8_t *fil;  // sample 16 (l % 16) of the span, channel 0
    int64_t nsamp;
    int c1, lane;
    i32x4 sel;
    i32x4 acc[TILES];

    // Channels c .. c + 3 (MASK: those below c1), their delays in lanes g .. of dl.
    template <bool MASK>
    __device__ __forceinline__ void group(int c, int g, int dl) {
        const int q = lane >> 4;
        const int dq = __shfl(dl, g + q);
        const bool live = !MASK || c + q < c1;  // (lanes past c1 hold the last channel's delay)
        const uint8_t *__restrict__ p = fil + int64_t(MASK ? min(c + q, c1 - 1) : c + q) * nsamp + dq;
        i32x4 b[TILES];
#pragma unroll
        for (int i = 0; i < TILES; ++i) __builtin_memcpy(&b[i], p + 256 * i, 16);  // one load from any byte address
#pragma unroll
        for (int i = 0; i < TILES; ++i) {
            b[i] ^= kFlip;
            if constexpr (MASK) b[i] = live ? b[i] : i32x4{0, 0, 0, 0};
            acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(sel, b[i], acc[i], 0, 0, 0);
        }
    }

    __device__ __forceinline__ void run(const Dispersion &disp, double kdm, int c0) {
        constexpr int UNR = TILES >= 4 ? 2 : 4;  // groups whose loads go out together
#pragma unroll
        for (int i = 0; i < TILES; ++i) acc[i] = i32x4{0, 0, 0, 0};
        for (; c0 < c1; c0 += 64) {
            const int dl = delay_fast(disp, kdm, min(c0 + lane, c1 - 1));  // of 64 channels at a time
            const int whole = min(64, c1 - c0) & ~3;
            int g = 0;
#pragma unroll 1
            for (; g + 4 * UNR <= whole; g += 4 * UNR) {
#pragma unroll
                for (int k = 0; k < UNR; ++k) group<false>(c0 + g + 4 * k, g + 4 * k, dl);
            }
#pragma unroll 1
            for (; g < whole; g += 4) group<false>(c0 + g, g, dl);
            if (whole < 64 && c0 + whole < c1) group<true>(c0 + whole, whole, dl);
        }
    }
};

template <int TILES, bool SPLIT>
__global__ __launch_bounds__(64 * DD_WAVES) void k_dedisperse(const uint8_t *__restrict__ fil, int nchan, int64_t nsamp,
                                                              Dispersion disp, int ndm, int64_t nout, Items items,
                                                              float *__restrict__ out) {
    constexpr int SPAN = 256 * TILES;
    const int64_t u = items.mine();
    if (u >= items.end) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ngrp = SPLIT ? ndm : (ndm + DD_WAVES - 1) / DD_WAVES;
    const int64_t span = u / ngrp;
    const int dm = SPLIT ? int(u - span * ngrp) : int(u - span * ngrp) * DD_WAVES + wave;
    if (!SPLIT && dm >= ndm) return;
    const int64_t first = span * SPAN, t0 = span_start(first, SPAN, nout);
    const int share = SPLIT ? (nchan + 4 * DD_WAVES - 1) / (4 * DD_WAVES) * 4 : nchan;  // whole groups of 4
    const int c0 = SPLIT ? min(nchan, wave * share) : 0;
    ChannelSums<TILES> s{fil + t0 + 16 * (lane & 15), nsamp, min(nchan, c0 + share), lane, one_at(lane & 15), {}};
    s.run(disp, disp.kdm[dm], c0);
    if constexpr (SPLIT) {
        __shared__ i32x4 part[DD_WAVES - 1][TILES][64];
        if (wave > 0) {
#pragma unroll
            for (int i = 0; i < TILES; ++i) part[wave - 1][i][lane] = s.acc[i];
        }
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int w = 0; w < DD_WAVES - 1; ++w)
#pragma unroll
            for (int i = 0; i < TILES; ++i) s.acc[i] += part[w][i][lane];
    }
    float *__restrict__ o = out + int64_t(dm) * nout;
#pragma unroll
    for (int i = 0; i < TILES; ++i)
        store_sums(o, t0 + 256 * i + 16 * (lane & 15) + 4 * (lane >> 4), first, s.acc[i] + 128 * nchan);
}

// A series shorter than the smallest span: one thread per output sample.
__global__ __launch_bounds__(256) void k_dedisperse_short(const uint8_t *__restrict__ fil, int nchan, int64_t nsamp,
                                                          Dispersion disp, int nout, float *__restrict__ out) {
    const int t = threadIdx.x;
    if (t >= nout) return;
    const double kdm = disp.kdm[blockIdx.x];
    uint32_t sum = 0;
    for (int c = 0; c < nchan; ++c) sum += fil[int64_t(c) * nsamp + t + delay_of(disp, kdm, c)];
    out[int64_t(blockIdx.x) * nout + t] = float(sum);
}

template <int TILES, bool SPLIT>
hipError_t launch_spans(const uint8_t *fil, int nchan, int64_t nsamp, const Dispersion &disp, int ndm, int64_t nout,
                        float *out, hipStream_t st) {
    const int64_t spans = (nout + 256 * TILES - 1) / (256 * TILES);
    const int64_t total = spans * (SPLIT ? ndm : (ndm + DD_WAVES - 1) / DD_WAVES);
    return launch_items(total, 64 * DD_WAVES, [&](unsigned grid, Items items) {
        hipLaunchKernelGGL((k_dedisperse<TILES, SPLIT>), dim3(grid), dim3(64 * DD_WAVES), 0, st, fil, nchan, nsamp, disp,
                           ndm, nout, items, out);
    });
}

// Row bytes of the LDS form for these trials: the span and one more piece, the
// largest spread of a group's delays (at most two samples above that at the
// lowest channel, whose delays differ most) and the bytes before the first
// aligned word.
int64_t lds_row(const Dispersion &disp, int nchan, int ndm) {
    int64_t spread = 0;
    for (int i = 0; i < ndm; i += DL_GROUP) {
        const double *k = disp.kdm + i;
        const auto mm = std::minmax_element(k, k + std::min(DL_GROUP, ndm - i));
        spread = std::max<int64_t>(spread, int64_t(delay_of(disp, *mm.second, nchan - 1)) - delay_of(disp, *mm.first, nchan - 1));
    }
    return (DL_SPAN + 16 + spread + 2 + 3 + 15) / 16 * 16;
}

hipError_t launch_trials(const uint8_t *fil, int nchan, int64_t nsamp, const Dispersion &disp, int ndm, int64_t nout,
                         float *out, hipStream_t st) {
    if (nout < 256) {
        hipLaunchKernelGGL(k_dedisperse_short, dim3(unsigned(ndm)), dim3(256), 0, st, fil, nchan, nsamp, disp,
                           int(nout), out);
        return hipGetLastError();
    }
    // The LDS form while the trials are close enough together for its rows.
    // Its time hardly depends on how many trials a group has nor, up to the 256
    // workgroups that run at once, on how many spans there are; that of the
    // direct forms is proportional to both.  Groups of ten trials and more
    // cross at about 2048 spans times trials (staged and direct, 64 channels:
    // 16 trials, 100 spans 35.8 us and 33.5, 120 spans 36.2 and 36.4, 160 spans
    // 36.4 and 41.2; 33 trials, 60 spans 36.4 and 36.6; 10 trials, 205 spans
    // 35.8 and 36.5; 257 channels, 16 trials, 120 spans 85.9 and 79.9, 140
    // spans 85.8 and 89.6).  Groups half empty, whose waves are half idle, cross
    // only with several workgroups a compute unit (257 channels: 8 trials, 205
    // spans 84.9 and 70.4, 410 spans 105.7 and 133.8; 7 trials, 520 spans 157.9
    // and 122.7, 1000 spans 205 and 260).
    const int64_t spans = (nout + DL_SPAN - 1) / DL_SPAN, groups = (ndm + DL_GROUP - 1) / DL_GROUP;
    const int64_t least = ndm >= 10 * groups ? 2048 : ndm >= 8 * groups ? 3200 : 7000;
    const int64_t row = lds_row(disp, nchan, ndm);
    if (nout >= DL_SPAN && ndm >= 7 && spans * ndm >= least && row <= DL_MAX_ROW) {
        const int64_t total = spans * groups;
        return launch_items(total, 64 * DL_WAVES, [&](unsigned grid, Items items) {
            hipLaunchKernelGGL(k_dedisperse_lds, dim3(grid), dim3(64 * DL_WAVES), size_t(2 * DL_CH * row), st, fil, nchan,
                               nsamp, disp, ndm, nout, int(row), items, out);
        });
    }
    // Otherwise spans of 1024 samples, a wave each, or spans of 256 with the
    // channels split over a workgroup's waves.  The split is for work too
    // small to give every SIMD several waves (512 channels, one trial of 2^16
    // samples: 24 us against 51; 257 channels, 33 trials of 60001: 65 against
    // 89) and for trials that do not fill workgroups (512 channels, 3 trials
    // of 2^22: 778 against 907); with few channels it leaves each wave too
    // little to do (16 channels, 3 trials of 2^22: 58 against 42).
    const int64_t waves = nout >= 1024 ? (nout / 1024) * ndm : 0;
    const bool wide = nchan < 64 ? waves >= 1024 : waves >= 4096 && (ndm % DD_WAVES == 0 || ndm > 16);
    return wide ? launch_spans<4, false>(fil, nchan, nsamp, disp, ndm, nout, out, st)
                : launch_spans<1, true>(fil, nchan, nsamp, disp, ndm, nout, out, st);
}

}  // namespace

hipError_t launch_dedisperse(const uint8_t *fil, int nchan, int64_t nsamp, double f_top, double foff, double tsamp,
                             const double *dms, int ndm, int64_t nout, float *out, hipStream_t st) {
    if (nchan <= 0 || ndm <= 0 || nout <= 0 || nsamp <= 0) return hipErrorInvalidValue;
    Dispersion disp;
    disp.f_top = f_top;
    disp.foff = foff;
    disp.inv_top2 = 1.0 / (f_top * f_top);
    disp.tsamp = tsamp;
    disp.inv_tsamp = 1.0 / tsamp;
    for (int i = 0; i < ndm; i += DD_LAUNCH_DMS) {
        const int n = std::min(DD_LAUNCH_DMS, ndm - i);
        for (int k = 0; k < DD_LAUNCH_DMS; ++k) disp.kdm[k] = k < n ? kDispersion * dms[i + k] : 0.0;
        const hipError_t e = launch_trials(fil, nchan, nsamp, disp, n, nout, out + int64_t(i) * nout, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace fdas
