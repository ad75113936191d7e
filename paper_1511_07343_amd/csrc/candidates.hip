// Candidate finishing on the device: order the harmonic-sum kernel's
// (unordered) records by (nharm, k, iz) and write the public records with r,
// z and the FP64 single-trial significance.  Lists of at most kFinishSmall
// records, nearly every trial's, take one kernel; longer ones an LSD radix
// sort (per 8-bit digit a count kernel and a scatter kernel that scans the
// counts itself).
// The record count stays on the device: every kernel reads it and clamps it
// to the buffer capacity, so nothing waits for the host in between.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/fdas.h"
#include "device_common.hpp"
#include "kernels.hpp"

namespace fdas {

namespace {

constexpr int RS_BLOCKS = 128;   // workgroups of the histogram and scatter passes
constexpr int RS_THREADS = 256;  // four waves
constexpr int RS_DIGITS = 256;   // 8-bit digits
constexpr int RS_AHEAD = 8;      // tiles of 256 records a scatter or count workgroup loads at once

__device__ __forceinline__ uint32_t clamp_count(const uint32_t *count, uint32_t cap) {
    const uint32_t c = *count;
    return c < cap ? c : cap;
}

__device__ __forceinline__ void block_range(uint32_t n, uint32_t &beg, uint32_t &end) {
    const uint32_t chunk = (n + RS_BLOCKS - 1) / RS_BLOCKS;
    beg = min(n, blockIdx.x * chunk);
    end = min(n, beg + chunk);
}

// Digit counts of a radix pass, block-major: hist[block * RS_DIGITS + digit]
// counts the records of `block`'s range (block_range) with that digit.

// key = (level nb + k) nz + iz, level = log2(nharm) in 0..4, k < nb, iz < nz:
// ascending keys are ascending (nharm, k, iz), and all keys are below
// 5 nb nz (32 bits, four 8-bit passes, at 2^23 samples and 201 templates).
__device__ __forceinline__ uint64_t cand_key(const DevCand &c, int64_t nb, int nz) {
    const uint64_t level = uint64_t(31 - __clz(c.nharm));
    return (level * uint64_t(nb) + uint64_t(uint32_t(c.k))) * uint64_t(nz) + uint64_t(uint32_t(c.iz));
}

// The drift (or acceleration) of plane row iz with two roundings, as the
// templates and trials are formed: a fused multiply-add would round once and
// can differ in the last bit.
__device__ __forceinline__ double row_value(const FinishArgs &a, int iz) {
#pragma clang fp contract(off)
    return a.td && a.nz == 1 ? 0.0 : -a.zmax + a.dz * double(iz);
}

// The public record of c.
__device__ __forceinline__ fdas_cand public_record(const DevCand &c, const FinishArgs &a) {
    fdas_cand o;
    o.k = c.k;
    o.iz = c.iz;
    o.nharm = c.nharm;
    o.r = double(c.k) / (double(c.nharm) * double(a.cpb));
    if (a.td) {
        o.z = row_value(a, c.iz) * o.r;
    } else {
        o.z = row_value(a, c.iz) / double(c.nharm);
    }
    o.power = c.power;
    o.sigma = float(significance_d(double(c.power), c.nharm));
    return o;
}

// Lists of at most kFinishSmall records: every workgroup takes FS_RECORDS of
// the records and ranks them among all keys, FS_TILE keys at a time in LDS, a
// quarter of them per wave, all lanes reading the same key (no two records
// share a key, so the ranks are the order); then it writes its records at
// their ranks.  One launch and no pass over memory in between: 130 records
// take 6 us, where a one-workgroup sort, seven empty radix kernels and the
// records' kernel took 40.  The work grows with the square of the list; from
// about 9000 records on the radix sort's launches and the host's wait for the
// counters in front of them are less (a search with 5000 records 65 us against
// 82 with the sort, 10000 records 91 against 86).
constexpr int FS_RECORDS = 64;
constexpr int FS_THREADS = 256;
constexpr int FS_TILE = 4096;

__global__ __launch_bounds__(FS_THREADS) void k_finish_small(FinishArgs a) {
    __shared__ __align__(16) uint64_t key[FS_TILE];
    __shared__ uint32_t less[FS_THREADS / 64][FS_RECORDS];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (a.count_dst && blockIdx.x == 0 && t < 6) a.count_dst[t] = a.count[t];
    const uint32_t n = clamp_count(a.count, a.cap), first = blockIdx.x * FS_RECORDS;
    if (n > kFinishSmall || first >= n) return;
    const uint32_t r = first + lane;
    const DevCand c = a.dc[min(r, n - 1)];
    const uint64_t mine = cand_key(c, a.nb, a.nz);
    uint32_t below = 0;
    for (uint32_t at = 0; at < n; at += FS_TILE) {
        const uint32_t m = min(n - at, uint32_t(FS_TILE));
        const uint32_t share = (m + 7) / 8 * 2;  // keys per wave, a whole number of pairs
        if (at > 0) __syncthreads();
        for (uint32_t i = t; i < 4 * share; i += FS_THREADS)
            key[i] = i < m ? cand_key(a.dc[at + i], a.nb, a.nz) : ~uint64_t(0);
        __syncthreads();
#pragma unroll 4
        for (uint32_t i = w * share; i < (w + 1) * share; i += 2) {
            const ulonglong2 k2 = *reinterpret_cast<const ulonglong2 *>(key + i);
            below += (k2.x < mine ? 1u : 0u) + (k2.y < mine ? 1u : 0u);
        }
    }
    less[w][lane] = below;
    __syncthreads();
    if (w != 0 || r >= n) return;
    const uint32_t rank = less[0][lane] + less[1][lane] + less[2][lane] + less[3][lane];
    if (rank < a.out_cap) a.out[rank] = public_record(c, a);
}

// The radix sort of longer lists.  One workgroup per block range (RS_BLOCKS of
// them): the keys and values of the range and the first pass's digit counts
// of the range.
__global__ __launch_bounds__(RS_THREADS) void k_cand_keys(const DevCand *__restrict__ dc, const uint32_t *__restrict__ count,
                                                          uint32_t cap, int64_t nb, int nz, uint64_t *__restrict__ keys,
                                                          uint32_t *__restrict__ vals, uint32_t *__restrict__ hist) {
    __shared__ uint32_t lh[RS_DIGITS];
    const uint32_t n = clamp_count(count, cap);
    if (n <= kFinishSmall) return;
    const int t = threadIdx.x;
    lh[t] = 0u;
    __syncthreads();
    uint32_t beg, end;
    block_range(n, beg, end);
    for (uint32_t i = beg + t; i < end; i += RS_THREADS) {
        const uint64_t key = cand_key(dc[i], nb, nz);
        keys[i] = key;
        vals[i] = i;
        atomicAdd(&lh[uint32_t(key) & (RS_DIGITS - 1u)], 1u);
    }
    __syncthreads();
    hist[blockIdx.x * RS_DIGITS + t] = lh[t];
}

// Digit counts of the pass at `shift` (passes after the first).
__global__ __launch_bounds__(RS_THREADS) void k_rs_hist(const uint64_t *__restrict__ keys,
                                                        const uint32_t *__restrict__ count, uint32_t cap, int shift,
                                                        uint32_t *__restrict__ hist) {
    __shared__ uint32_t lh[RS_DIGITS];
    const uint32_t n = clamp_count(count, cap);
    if (n <= kFinishSmall) return;
    const int t = threadIdx.x;
    lh[t] = 0u;
    __syncthreads();
    uint32_t beg, end;
    block_range(n, beg, end);
    for (uint32_t batch = beg; batch < end; batch += RS_AHEAD * RS_THREADS) {
        uint64_t kk[RS_AHEAD];
#pragma unroll
        for (int q = 0; q < RS_AHEAD; ++q) {
            const uint32_t i = batch + uint32_t(q) * RS_THREADS + t;
            kk[q] = i < end ? keys[i] : 0;
        }
#pragma unroll
        for (int q = 0; q < RS_AHEAD; ++q)
            if (batch + uint32_t(q) * RS_THREADS + t < end)
                atomicAdd(&lh[uint32_t(kk[q] >> shift) & (RS_DIGITS - 1u)], 1u);
    }
    __syncthreads();
    hist[blockIdx.x * RS_DIGITS + t] = lh[t];
}

// One pass of the LSD radix sort: a stable scatter of one 8-bit digit.
// Each workgroup first derives its output offsets from the pass's digit
// counts (digit t's total over all blocks and over the blocks before this
// one, then a scan of the totals over the digits); then it re-walks its range
// in tiles of 256 (one element per thread, element order = wave-major lane
// order): a lane's rank among same-digit lanes of its wave comes from 8
// ballots, wave offsets from LDS counts, and a running per-digit offset
// carries across tiles.
__global__ __launch_bounds__(RS_THREADS) void k_rs_pass(const uint64_t *__restrict__ kin,
                                                        const uint32_t *__restrict__ vin,
                                                        const uint32_t *__restrict__ count, uint32_t cap, int shift,
                                                        const uint32_t *__restrict__ hist, uint64_t *__restrict__ kout,
                                                        uint32_t *__restrict__ vout) {
    __shared__ uint32_t base[RS_DIGITS];
    __shared__ uint32_t cnt[RS_THREADS / 64][RS_DIGITS];
    __shared__ uint32_t wsum[RS_THREADS / 64];
    const uint32_t n = clamp_count(count, cap);
    if (n <= kFinishSmall) return;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint32_t before = 0, total = 0;
#pragma unroll 16
    for (int b = 0; b < RS_BLOCKS; ++b) {
        const uint32_t c = hist[b * RS_DIGITS + t];
        total += c;
        before += b < int(blockIdx.x) ? c : 0u;
    }
    uint32_t incl = total;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t off = incl - total + before;
    for (int ww = 0; ww < w; ++ww) off += wsum[ww];
    base[t] = off;  // ordered before its first use by the tile loop's barrier
    uint32_t beg, end;
    block_range(n, beg, end);
    const uint64_t lt_mask = (uint64_t(1) << lane) - 1;
    // RS_AHEAD tiles' keys and values are loaded together, so that the
    // tiles of a batch wait for memory once
    for (uint32_t batch = beg; batch < end; batch += RS_AHEAD * RS_THREADS) {
        uint64_t kk[RS_AHEAD];
        uint32_t vv[RS_AHEAD];
#pragma unroll
        for (int q = 0; q < RS_AHEAD; ++q) {
            const uint32_t i = batch + uint32_t(q) * RS_THREADS + t;
            kk[q] = i < end ? kin[i] : 0;
            vv[q] = i < end ? vin[i] : 0u;
        }
#pragma unroll
        for (int q = 0; q < RS_AHEAD; ++q) {
            const uint32_t tile = batch + uint32_t(q) * RS_THREADS;
            if (tile >= end) break;  // the same for every thread
#pragma unroll
            for (int ww = 0; ww < RS_THREADS / 64; ++ww) cnt[ww][t] = 0;
            __syncthreads();
            const uint32_t i = tile + t;
            const bool valid = i < end;
            const uint64_t key = kk[q];
            const uint32_t val = vv[q];
            const uint32_t d = valid ? uint32_t(key >> shift) & 255u : 0u;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t m = __ballot(valid && bit);
                peers &= bit ? m : ~m;
            }
            const uint32_t rank = __popcll(peers & lt_mask);
            if (valid && rank == 0) cnt[w][d] = __popcll(peers);
            __syncthreads();
            // thread t owns digit t: offsets of each wave within the tile
            uint32_t o = 0;
#pragma unroll
            for (int ww = 0; ww < RS_THREADS / 64; ++ww) {
                const uint32_t c = cnt[ww][t];
                cnt[ww][t] = o;
                o += c;
            }
            __syncthreads();
            if (valid) {
                const uint32_t pos = base[d] + cnt[w][d] + rank;
                kout[pos] = key;
                vout[pos] = val;
            }
            __syncthreads();
            base[t] += o;
        }
    }
}

// The public records of the first min(count, cap, out_cap) sorted records, and
// the counters where they are wanted.
__global__ __launch_bounds__(256) void k_cand_finalize(FinishArgs a, const uint32_t *__restrict__ order) {
    const uint32_t n = clamp_count(a.count, a.cap);
    if (n <= kFinishSmall) return;
    if (a.count_dst && blockIdx.x == 0 && threadIdx.x < 6) a.count_dst[threadIdx.x] = a.count[threadIdx.x];
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < min(n, a.out_cap); i += gridDim.x * blockDim.x)
        a.out[i] = public_record(a.dc[order[i]], a);
}

// min(count, cap) records, and the six counter words, written straight into
// page-locked host memory (device aliases), so that the host needs no round
// trip for the count before it can copy the records.
__global__ __launch_bounds__(256) void k_copy_records(const fdas_cand *__restrict__ src,
                                                      const uint32_t *__restrict__ count, uint32_t cap,
                                                      fdas_cand *__restrict__ dst, uint32_t *__restrict__ count_dst) {
    const uint32_t n = clamp_count(count, cap);
    const uint32_t words = n * uint32_t(sizeof(fdas_cand) / 4);
    const uint32_t *__restrict__ s = reinterpret_cast<const uint32_t *>(src);
    uint32_t *__restrict__ d = reinterpret_cast<uint32_t *>(dst);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < words; i += gridDim.x * blockDim.x) d[i] = s[i];
    if (blockIdx.x == 0 && threadIdx.x < 6) count_dst[threadIdx.x] = count[threadIdx.x];
}

}  // namespace

hipError_t launch_copy_records(const fdas_cand *src, const uint32_t *count, uint32_t cap, fdas_cand *dst,
                               uint32_t *count_dst, hipStream_t st) {
    static_assert(sizeof(fdas_cand) % 4 == 0, "whole words");
    const uint64_t words = uint64_t(cap) * (sizeof(fdas_cand) / 4);
    const uint64_t blocks = (words + 255) / 256;
    const unsigned grid = unsigned(blocks < 1024 ? (blocks > 0 ? blocks : 1) : 1024);
    hipLaunchKernelGGL(k_copy_records, dim3(grid), dim3(256), 0, st, src, count, cap, dst, count_dst);
    return hipGetLastError();
}

// Layout: keys k0, k1 (cap each), values v0, v1 (cap each), then the digit
// counts at the next 16-byte boundary.
size_t cand_sort_scratch_bytes(uint32_t cap) {
    return size_t(cap) * (2 * sizeof(uint64_t) + 2 * sizeof(uint32_t)) + 16 + size_t(RS_DIGITS) * RS_BLOCKS * 4;
}

hipError_t launch_finish_small(const FinishArgs &a, hipStream_t st) {
    const uint32_t most = a.cap < kFinishSmall ? a.cap : kFinishSmall;
    const unsigned grid = most > 0 ? (most + FS_RECORDS - 1) / FS_RECORDS : 1;
    hipLaunchKernelGGL(k_finish_small, dim3(grid), dim3(FS_THREADS), 0, st, a);
    return hipGetLastError();
}

// Launches: keys (with the first pass's counts), per radix pass the digit
// counts (after the first) and the scatter, the public records.  Each returns
// at once for lists that launch_finish_small has finished.
hipError_t launch_finish_large(const FinishArgs &a, void *scratch, hipStream_t st) {
    const uint32_t cap = a.cap;
    if (cap <= kFinishSmall) return hipSuccess;
    const uint64_t span = 5 * uint64_t(a.nb) * uint64_t(a.nz);  // keys are below this
    int bits = 1;
    while (bits < 64 && (uint64_t(1) << bits) < span) ++bits;
    const int passes = (bits + 7) / 8;
    uint64_t *k0 = static_cast<uint64_t *>(scratch);
    uint64_t *k1 = k0 + cap;
    uint32_t *v0 = reinterpret_cast<uint32_t *>(k1 + cap);
    uint32_t *v1 = v0 + cap;
    uint32_t *hist = reinterpret_cast<uint32_t *>((reinterpret_cast<uintptr_t>(v1 + cap) + 15) & ~uintptr_t(15));
    const uint64_t blocks = (uint64_t(cap) + 255) / 256;
    // Into host memory the records leave at the PCIe rate: with fewer
    // threads than records (about two each for 241 k records) a wave's writes
    // of one record go out while it computes its next significance, instead
    // of every significance first and then all the writes (about 12 us less).
    const uint64_t gmax = a.to_host ? 512 : 1024;
    const unsigned grid = unsigned(blocks < gmax ? blocks : gmax);
    hipLaunchKernelGGL(k_cand_keys, dim3(RS_BLOCKS), dim3(RS_THREADS), 0, st, a.dc, a.count, cap, a.nb, a.nz, k0, v0,
                       hist);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int p = 0; p < passes; ++p) {
        if (p > 0)
            hipLaunchKernelGGL(k_rs_hist, dim3(RS_BLOCKS), dim3(RS_THREADS), 0, st, k0, a.count, cap, 8 * p, hist);
        hipLaunchKernelGGL(k_rs_pass, dim3(RS_BLOCKS), dim3(RS_THREADS), 0, st, k0, v0, a.count, cap, 8 * p, hist, k1,
                           v1);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        uint64_t *tk = k0;
        k0 = k1;
        k1 = tk;
        uint32_t *tv = v0;
        v0 = v1;
        v1 = tv;
    }
    hipLaunchKernelGGL(k_cand_finalize, dim3(grid), dim3(256), 0, st, a, v0);
    return hipGetLastError();
}

}  // namespace fdas
