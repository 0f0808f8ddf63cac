// Device-wide exclusive prefix sums of uint32 arrays, the parts shared by the
// kernels that scan (scan.hip, and the stages that do more with the prefix of
// an element than store it).
//
// A scan is two launches: the sums of tiles of kScanTile elements, and a pass
// over the tiles that adds up the sums of the tiles before its own (every
// workgroup by itself: at kDirectTiles tiles an average workgroup reads 8 KB
// that lie in L2).  Launching costs more than reading here: a scan with its
// own launch for the tile sums' scan took 12 us on 2.6e5 elements against 8.
// Beyond kDirectTiles one workgroup scans the tile sums in between.
// LDS indices are padded by one word per 32 to keep the per-thread runs of 16
// words off a single bank.
#pragma once

#include "hf_internal.h"

namespace hf {

constexpr int kScanItems = 16;                    // elements per thread
constexpr int kScanTile = kBlock * kScanItems;    // elements per tile
constexpr int64_t kDirectTiles = 4096;
constexpr int kScanLds = kScanTile + kScanTile / 32;

inline int64_t scan_tiles(int64_t n) { return n > 0 ? (n + kScanTile - 1) / kScanTile : 1; }

__device__ __forceinline__ int scan_pad(int i) { return i + (i >> 5); }

// Exclusive scan of one value per thread across an NT-thread block; *total
// receives the block sum.
template <int NT = kBlock>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *total) {
    __shared__ uint32_t wsum[NT / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t inc = wave_incl_scan(v);
    if (lane == 63) wsum[wid] = inc;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; k++) {
        if (k < wid) pre += wsum[k];
        tot += wsum[k];
    }
    __syncthreads();
    *total = tot;
    return pre + inc - v;
}

// Sum of one value per thread across the kBlock threads, returned to all.
__device__ __forceinline__ uint32_t block_sum(uint32_t v) {
    __shared__ uint32_t bsum[kBlock / 64];
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if ((threadIdx.x & 63) == 0) bsum[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t t = 0;
#pragma unroll
    for (int k = 0; k < kBlock / 64; k++) t += bsum[k];
    __syncthreads();
    return t;
}

// The offset of tile t: its entry of the scanned tile sums, or the sum of the
// entries before it.
__device__ __forceinline__ uint32_t tile_offset(const uint32_t *__restrict__ sums, uint32_t t, bool scanned) {
    if (scanned) return sums[t];
    uint32_t s = 0;
    for (uint32_t k = threadIdx.x; k < t; k += 4 * kBlock) {
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) s += k + u * kBlock < t ? sums[k + u * kBlock] : 0u;
    }
    return block_sum(s);
}

// The tile's elements into LDS (16-byte loads where the tile is whole: `in` is
// 16-byte aligned), then kScanItems consecutive ones per thread into v.
template <class Val>
__device__ __forceinline__ void tile_load(const uint32_t *__restrict__ in, int64_t base, int64_t n, uint32_t *buf,
                                          uint32_t (&v)[kScanItems], Val val) {
    if (base + kScanTile <= n) {
        const uint4 *p = reinterpret_cast<const uint4 *>(in + base);
#pragma unroll
        for (int k = 0; k < kScanItems / 4; k++) {
            const int q = k * kBlock + threadIdx.x;
            const uint4 x = p[q];
            buf[scan_pad(4 * q + 0)] = val(x.x);
            buf[scan_pad(4 * q + 1)] = val(x.y);
            buf[scan_pad(4 * q + 2)] = val(x.z);
            buf[scan_pad(4 * q + 3)] = val(x.w);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; k++) {
            const int idx = k * kBlock + threadIdx.x;
            buf[scan_pad(idx)] = base + idx < n ? val(in[base + idx]) : 0u;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanItems; k++) v[k] = buf[scan_pad(threadIdx.x * kScanItems + k)];
}

// f(element) over the tile's elements in [base, n), this thread's share.
template <class F>
__device__ __forceinline__ void tile_each(const uint32_t *__restrict__ in, int64_t base, int64_t n, F f) {
    if (base + kScanTile <= n) {
        const uint4 *p = reinterpret_cast<const uint4 *>(in + base);
#pragma unroll
        for (int k = 0; k < kScanItems / 4; k++) {
            const uint4 x = p[k * kBlock + threadIdx.x];
            f(x.x);
            f(x.y);
            f(x.z);
            f(x.w);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; k++) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            if (i < n) f(in[i]);
        }
    }
}

// Exclusive scan of the tile sums in place, where there are more than
// kDirectTiles of them (`arrays` runs of `tiles` words, `stride` words apart);
// returns whether they are scanned now.
bool scan_sums(uint32_t *sums, int64_t tiles, int64_t stride, int arrays, hipStream_t s);

}  // namespace hf
