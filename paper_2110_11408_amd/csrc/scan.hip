// Device-wide exclusive prefix sums of uint32 arrays (scan_tile.h), fill kernels
// and the read-back of device words.
//
// (A single pass with decoupled look-back was slower here: on this chip the
// chain of status words between thousands of tiles goes through memory that
// every XCD must see, a few microseconds per link.)
#include "hf_internal.h"
#include "scan_tile.h"

namespace hf {

namespace {

// What is scanned: the values, or the set bits of every word.
template <bool kBits>
__device__ __forceinline__ uint32_t scan_val(uint32_t x) { return kBits ? (uint32_t)__popc(x) : x; }

template <bool kBits>
__global__ __launch_bounds__(kBlock) void k_tile_sums(const uint32_t *__restrict__ in, int64_t n,
                                                      uint32_t *__restrict__ sums) {
    uint32_t s = 0;
    tile_each(in, (int64_t)blockIdx.x * kScanTile, n, [&](uint32_t x) { s += scan_val<kBits>(x); });
    const uint32_t tot = block_sum(s);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

template <bool kBits>
__global__ __launch_bounds__(kBlock) void k_tile_scan(const uint32_t *__restrict__ in,
                                                      uint32_t *__restrict__ out, int64_t n,
                                                      const uint32_t *__restrict__ sums, bool scanned) {
    __shared__ uint32_t buf[kScanLds];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t v[kScanItems];
    tile_load(in, base, n, buf, v, scan_val<kBits>);
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) s += v[k];
    uint32_t tot;
    uint32_t run = block_excl_scan(s, &tot);
    const uint32_t toff = blockIdx.x > 0 ? tile_offset(sums, blockIdx.x, scanned) : 0u;
    run += toff;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        buf[scan_pad(threadIdx.x * kScanItems + k)] = run;
        run += v[k];
    }
    __syncthreads();
    if (base + kScanTile <= n) {
        uint4 *p = reinterpret_cast<uint4 *>(out + base);
#pragma unroll
        for (int k = 0; k < kScanItems / 4; k++) {
            const int q = k * kBlock + threadIdx.x;
            p[q] = make_uint4(buf[scan_pad(4 * q + 0)], buf[scan_pad(4 * q + 1)], buf[scan_pad(4 * q + 2)],
                              buf[scan_pad(4 * q + 3)]);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; k++) {
            const int idx = k * kBlock + threadIdx.x;
            const int64_t i = base + idx;
            if (i < n) out[i] = buf[scan_pad(idx)];
        }
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = toff + tot;
}

// Exclusive scan of `tiles` words in place by one workgroup (one array of
// `stride` words per workgroup).
constexpr int kSumsThreads = 1024;
__global__ __launch_bounds__(kSumsThreads) void k_sums_scan(uint32_t *__restrict__ sums, int64_t tiles,
                                                            int64_t stride) {
    uint32_t *p = sums + (int64_t)blockIdx.x * stride;
    uint32_t run = 0;
    for (int64_t t0 = 0; t0 < tiles; t0 += kSumsThreads * kScanItems) {
        const int64_t b = t0 + (int64_t)threadIdx.x * kScanItems;
        uint32_t v[kScanItems], s = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; k++) {
            v[k] = b + k < tiles ? p[b + k] : 0u;
            s += v[k];
        }
        uint32_t tot;
        uint32_t at = run + block_excl_scan<kSumsThreads>(s, &tot);
#pragma unroll
        for (int k = 0; k < kScanItems; k++) {
            if (b + k < tiles) p[b + k] = at;
            at += v[k];
        }
        run += tot;
    }
}

__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t *p, uint32_t v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// 16-byte stores for a 16-byte-aligned array of n4 words x4, then the tail.
__global__ __launch_bounds__(kBlock) void k_fill_u32x4(uint4 *p, uint32_t v, int64_t n4, uint32_t *tail,
                                                       int ntail) {
    const uint4 q = make_uint4(v, v, v, v);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = q;
    if (blockIdx.x == 0 && (int)threadIdx.x < ntail) tail[threadIdx.x] = v;
}

// Copies k device words into pinned host memory with system-scope stores, so
// the host sees them once the stream has drained.
__global__ void k_publish(WordSrc src, int k, uint32_t *host, uint64_t *clock) {
    stamp(clock);
    const int t = threadIdx.x;
    if (t < k) __hip_atomic_store(host + t, *src.p[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(kBlock) void k_begin(BeginCopy c, int32_t *counters, int32_t *err, uint64_t *clock) {
    stamp(clock);
    const uint32_t t0 = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    const uint32_t *src = c.src;
    for (int a = 0; a < 4; a++) {
        for (uint32_t i = t0; i < c.words[a]; i += step) c.dst[a][i] = src[i];
        src += c.words[a];
    }
    if (t0 < 16) counters[t0] = 0;
    if (t0 < 2) err[t0] = t0 ? 0x7fffffff : 0;
}

int64_t grid_for(int64_t n, int64_t cap = 1 << 20) {
    int64_t b = (n + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    return b < cap ? b : cap;
}

}  // namespace

void fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    if ((reinterpret_cast<uintptr_t>(p) & 15u) == 0 && n >= 1024) {
        const int64_t n4 = n / 4;
        hipLaunchKernelGGL(k_fill_u32x4, dim3(grid_for(n4)), dim3(kBlock), 0, s, reinterpret_cast<uint4 *>(p), v, n4,
                           p + 4 * n4, (int)(n - 4 * n4));
        return;
    }
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n)), dim3(kBlock), 0, s, p, v, n);
}

void fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
    fill_u32(reinterpret_cast<uint32_t *>(p), (uint32_t)v, n, s);
}

hipError_t begin_call(const BeginCopy &c, int32_t *counters, int32_t *err, uint64_t *clock, hipStream_t s) {
    const int64_t words = (int64_t)c.words[0] + c.words[1] + c.words[2] + c.words[3];
    hipLaunchKernelGGL(k_begin, dim3(grid_for(words, 64)), dim3(kBlock), 0, s, c, counters, err, clock);
    return hipGetLastError();
}

hipError_t publish_words(const WordSrc &src, int k, uint32_t *host, hipStream_t s, uint64_t *clock) {
    if (k < 0 || k > WordSrc::kMax) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, src, k, host, clock);
    return hipGetLastError();
}

void collect_words(const uint32_t *host, int k, uint32_t *out) {
    for (int i = 0; i < k; i++) out[i] = __atomic_load_n(host + i, __ATOMIC_ACQUIRE);
}

hipError_t read_words(const WordSrc &src, int k, uint32_t *host, uint32_t *out, hipStream_t s, uint64_t *clock) {
    hipError_t e = publish_words(src, k, host, s, clock);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    collect_words(host, k, out);
    return hipSuccess;
}

bool scan_sums(uint32_t *sums, int64_t tiles, int64_t stride, int arrays, hipStream_t s) {
    if (tiles <= kDirectTiles) return false;
    hipLaunchKernelGGL(k_sums_scan, dim3((unsigned)arrays), dim3(kSumsThreads), 0, s, sums, tiles, stride);
    return true;
}

// Tile sums of the longest scans: of four quantities at once over the binning's
// tiles, two over the keys, and one over the radix counts.
int64_t scan_tmp_words(int64_t n) {
    const int64_t bin = 4 * bin_tiles(n), keys = 2 * scan_tiles(n), counts = scan_tiles(radix_hist_len(n));
    return (bin > keys ? (bin > counts ? bin : counts) : (keys > counts ? keys : counts)) + 16;
}

template <bool kBits>
static void scan_impl(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp, hipStream_t s) {
    const int64_t tiles = scan_tiles(n);
    bool scanned = false;
    if (tiles > 1) {
        hipLaunchKernelGGL(k_tile_sums<kBits>, dim3(tiles), dim3(kBlock), 0, s, in, n, tmp);
        scanned = scan_sums(tmp, tiles, tiles, 1, s);
    }
    hipLaunchKernelGGL(k_tile_scan<kBits>, dim3(tiles), dim3(kBlock), 0, s, in, out, n, tmp, scanned);
}

void scan_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp, hipStream_t s) {
    scan_impl<false>(in, out, n, tmp, s);
}

void scan_bits_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp, hipStream_t s) {
    scan_impl<true>(in, out, n, tmp, s);
}

}  // namespace hf
