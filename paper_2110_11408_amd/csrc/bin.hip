// Cell binning: a stable sort of the particles by (cell, sub-cell), ties in
// original index order.
//
// The paper's host code receives particles already ordered by cell from the
// N-body engine (Sec. 2.3.4); here the caller hands over an unordered float32
// [n][3] array, so the library builds the order itself:
//   1. key = cell * k^3 + sub-cell per particle (range check of the input), and
//      the digit counts of the first pass on the way;
//   2. the keys are put into buckets by their top bits, and a workgroup per
//      bucket (several for a long one) sorts it by the other bits in LDS and
//      writes the sorted records.
//      Up to kPartitionMost particles one pass over (key, index) words makes
//      up to 1024 buckets; beyond, two passes make up to 2^18, and carry the
//      positions with them, so that nothing is gathered from the unordered
//      input.  (A least-significant-digit radix sort over all digits remains
//      for what neither takes, see sort_plan, and for the later stages' lists.)
//      A pass over a digit: a block counts the digits of its tile of 2048
//      consecutive elements; an exclusive scan of the digit-major [digit][tile]
//      counts gives every (digit, tile) its output offset; the tile is then
//      walked again in order, each element's rank among equal digits coming
//      from the ballots of its digit bits (lower lanes first), so the pass is
//      stable, and written out through LDS in digit order (coalesced runs).
//      Consecutive tiles run on one XCD, so the runs that consecutive tiles
//      write for a digit (adjacent in the output) meet in one L2;
//   3. the sorted order writes two float4 streams per particle:
//        spos = (x, y, z, original index bits)    -- the paper's float quad with
//               the index stored bitwise (Sec. 2.3.3), used by FP64 predicates;
//        sloc = (x, y, z relative to the cell corner, in units of b; cell id
//               bits) -- FP32 coordinates whose differences across a periodic
//               face stay exact, used by the density loop and prefilters;
//   4. the cell index: a bit per cell that holds particles, the number of the
//      first one per 32 cells, and every such cell's first particle, written with
//      the lists of the dense chunks and sparse particles.
// Cells are at least max(b, l) wide; each is split into k^3 sub-cells whose
// diagonal is below l, so all particles of one sub-cell are friends.  The
// boxes of one call are binned together: their cells are numbered box after
// box, so the sorted order is box-major and box b keeps the slots of its
// input range.
//
// Work decomposition shared by the neighbour-loop kernels: a cell holding at
// least kDenseMin particles is "dense".  Dense cells get a table of their
// sub-cell offsets and are cut into chunks of at most 64 consecutive particles
// (one wavefront each); particles of the other cells form the "sparse" list
// (one thread each).  The in-cell order, and therefore every summation order,
// is fixed by the data, never by thread scheduling.
#include <stdlib.h>

#include "hf_internal.h"
#include "scan_tile.h"

namespace hf {

namespace {

inline int64_t blocks(int64_t n) { return (n + kBlock - 1) / kBlock; }

__device__ __forceinline__ int cell_coord(float x, const Geo &g) {
    int c = (int)floor((double)x * g.inv_cell);
    return c < 0 ? 0 : (c >= g.nc ? g.nc - 1 : c);
}

__device__ __forceinline__ int sub_coord(float x, int c, const Geo &g) {
    int s = (int)floor(((double)x - (double)c * g.cell) * g.inv_sub);
    return s < 0 ? 0 : (s >= g.ksub ? g.ksub - 1 : s);
}

// Cell and sub-cell of a position of box g, and the sort key made of them.
struct Spot {
    int cx, cy, cz;
    uint32_t c, sub;  // cell in the call's numbering, sub-cell
    uint64_t key;     // c * nsub_max + sub
};
__device__ __forceinline__ Spot spot_of(const Geo &g, int nsub_max, float x, float y, float z) {
    Spot p;
    p.cx = cell_coord(x, g);
    p.cy = cell_coord(y, g);
    p.cz = cell_coord(z, g);
    p.c = g.cell_base + ((uint32_t)p.cz * (uint32_t)g.nc + (uint32_t)p.cy) * (uint32_t)g.nc + (uint32_t)p.cx;
    const int k = g.ksub;
    p.sub = (uint32_t)((sub_coord(z, p.cz, g) * k + sub_coord(y, p.cy, g)) * k + sub_coord(x, p.cx, g));
    p.key = (uint64_t)p.c * (uint64_t)nsub_max + p.sub;
    return p;
}

__device__ __forceinline__ bool inside(const Geo &g, float x, float y, float z) {
    const float Lf = (float)g.L;
    return x >= 0.0f && x < Lf && y >= 0.0f && y < Lf && z >= 0.0f && z < Lf;
}

// Sort key of particle i: cell * nsub_max + sub-cell, the cell numbered in the
// call's numbering (box after box).  Packed mode stores (key << ib) | i in one
// word (ib bits hold the index); otherwise the index travels in a separate
// payload array.
constexpr int kRadixMaxBits = 8;                    // digits of a pass of the radix sort
constexpr int kPartBits = 10;                       // digits of the partition pass
constexpr int kRadixWaves = 4;                      // wavefronts per tile
constexpr int kRadixIters = 8;                      // 64-element steps per wavefront
// 2048 elements per tile: the scatter's LDS tile (16 KB of keys) then lets
// seven blocks share a CU, twice as many as with 4096
constexpr int64_t kTile = 64 * kRadixWaves * kRadixIters;

// Digit counts of a tile, stored digit-major ([digit][tile]), with one LDS
// atomic per element: equal digits in a wavefront cost an LDS cycle each, fewer
// than the ballots of the digit bits that find them (the counts were bound by
// the vector ALU, 38 us a pass on 1.7e7 keys).
__device__ __forceinline__ void counts_out(const uint32_t *h, int nd, int64_t t, int64_t ntiles,
                                           uint32_t *__restrict__ hist) {
    __syncthreads();
    for (int d = threadIdx.x; d < nd; d += 256) hist[(int64_t)d * ntiles + t] = h[d];
}

// A workgroup keys one tile (eight particles per thread, their positions loaded
// together: one load in flight per thread leaves most of the bandwidth unused)
// and counts its digits [shift, shift + D) for the first pass.
__global__ __launch_bounds__(256) void k_bin_key(const float *__restrict__ pos, int64_t n, Boxes bx, int ib,
                                                 uint64_t *__restrict__ key, int shift, int D, int64_t ntiles,
                                                 uint32_t *__restrict__ hist, int32_t *__restrict__ err) {
    __shared__ uint32_t h[1 << kPartBits];
    const int64_t t = xcd_block();
    const int nd = 1 << D;
    for (int d = threadIdx.x; d < nd; d += 256) h[d] = 0u;
    const int64_t i0 = t * kTile + threadIdx.x;
    float px[kRadixIters], py[kRadixIters], pz[kRadixIters];
#pragma unroll
    for (int u = 0; u < kRadixIters; u++) {
        const int64_t i = i0 + (int64_t)u * 256;
        px[u] = i < n ? pos[3 * i + 0] : 0.0f;
        py[u] = i < n ? pos[3 * i + 1] : 0.0f;
        pz[u] = i < n ? pos[3 * i + 2] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRadixIters; u++) {
        const int64_t i = i0 + (int64_t)u * 256;
        if (i >= n) break;
        const int box = box_of(bx, (uint32_t)i);
        const Geo &g = bx.geo[box];
        if (!inside(g, px[u], py[u], pz[u])) flag_error(err, 1, box);
        const uint64_t kk = spot_of(g, bx.nsub_max, px[u], py[u], pz[u]).key;
        const uint64_t kw = ib > 0 ? (kk << ib) | (uint64_t)i : kk;
        key[i] = kw;
        atomicAdd(&h[(uint32_t)(kw >> shift) & (uint32_t)(nd - 1)], 1u);
    }
    counts_out(h, nd, t, ntiles, hist);
}

// Lanes holding the same D-bit digit as this lane (within `active`).
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, int D, uint64_t active) {
    uint64_t m = active;
    for (int b = 0; b < D; b++) {
        const uint64_t bal = __ballot((d >> b) & 1u);
        m &= ((d >> b) & 1u) ? bal : ~bal;
    }
    return m;
}

__device__ __forceinline__ uint64_t lanes_below(int lane) {
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Digit counts of one tile, all its elements loaded before counting.
__global__ __launch_bounds__(256) void k_radix_count(const uint64_t *__restrict__ key, int64_t n, int shift,
                                                     int D, int64_t ntiles, uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[1 << kRadixMaxBits];
    const int64_t t = xcd_block();
    const int nd = 1 << D;
    for (int d = threadIdx.x; d < nd; d += 256) h[d] = 0u;
    const int64_t base = t * kTile + threadIdx.x;
    uint64_t k[kRadixIters];
#pragma unroll
    for (int it = 0; it < kRadixIters; it++) {
        const int64_t e = base + it * 256;
        k[it] = e < n ? key[e] : 0ull;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRadixIters; it++)
        if (base + it * 256 < n) atomicAdd(&h[(uint32_t)(k[it] >> shift) & (uint32_t)(nd - 1)], 1u);
    counts_out(h, nd, t, ntiles, hist);
}

// Block-wide exclusive scan of one value per thread (NW wavefronts).
template <int NW = kRadixWaves>
__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t *s_tot) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = v;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
    }
    if (lane == 63) s_tot[w] = inc;
    __syncthreads();
    uint32_t pre = 0;
#pragma unroll
    for (int x = 0; x < NW; x++) pre += x < w ? s_tot[x] : 0u;
    return pre + inc - v;
}

// An element's place among the equal digits of its 64-element step: how many
// before it (bits 0-7), how many in all (8-15), whether it is the first (16).
// Kept from the counting walk for the ranking one: finding the peers again
// made the scatter bound by the vector ALU (78 us a pass on 1.7e7 keys).
__device__ __forceinline__ uint32_t step_place(uint32_t d, int D, bool act) {
    const uint64_t m = digit_peers(d, D, __ballot(act));
    const uint32_t before = (uint32_t)__popcll(m & lanes_below((int)(threadIdx.x & 63)));
    return before | ((uint32_t)__popcll(m) << 8) | (before == 0u ? 1u << 16 : 0u);
}

// Counts per wavefront and digit (o[w][d]) to the first place of each in the
// digit order of the tile, which starts at 0; lstart[d] receives the digit's
// start.  nd <= threads * PER digits, PER consecutive ones each.
template <int PER, int NW = kRadixWaves, class Row>
__device__ __forceinline__ void digit_starts(Row o, int nd, uint32_t *lstart, uint32_t *s_tot) {
    const int d0 = (int)threadIdx.x * PER;
    uint32_t tot[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; q++) {
        tot[q] = 0;
        if (d0 + q < nd)
            for (int x = 0; x < NW; x++) tot[q] += o[x][d0 + q];
        sum += tot[q];
    }
    uint32_t at = block_scan_excl<NW>(sum, s_tot);
#pragma unroll
    for (int q = 0; q < PER; q++) {
        if (d0 + q < nd) {
            lstart[d0 + q] = at;
            uint32_t b = at;
            for (int x = 0; x < NW; x++) {
                const uint32_t c = o[x][d0 + q];
                o[x][d0 + q] = b;
                b += c;
            }
        }
        at += tot[q];
    }
}

// Stable scatter of one tile.  Every element's position inside the tile's
// digit-sorted order is its digit's start in the tile plus the count of equal
// digits before it (earlier wavefronts, earlier steps, lower lanes); the tile
// is first placed in LDS in that order and then written out in order, so
// consecutive threads write consecutive addresses of one digit's run (the
// digit's global offset for this tile comes from the scanned counts).
template <bool kPacked, int kBits>
__global__ __launch_bounds__(256) void k_radix_scatter(const uint64_t *__restrict__ kin,
                                                       const uint32_t *__restrict__ vin, int64_t n, int shift,
                                                       int D, int64_t ntiles, const uint32_t *__restrict__ hscan,
                                                       uint64_t *__restrict__ kout, uint32_t *__restrict__ vout) {
    constexpr int kPer = (1 << kBits) > 256 ? (1 << kBits) / 256 : 1;
    __shared__ uint32_t o[kRadixWaves][1 << kBits];
    __shared__ uint32_t lstart[1 << kBits];
    __shared__ uint32_t s_tot[kRadixWaves];
    __shared__ uint64_t sk[kTile];
    __shared__ uint32_t sv[kPacked ? 1 : kTile];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, tid = threadIdx.x;
    const int64_t t = xcd_block();
    const int nd = 1 << D;
    const uint32_t dmask = (uint32_t)(nd - 1);
    for (int d = lane; d < nd; d += 64) o[w][d] = 0u;
    const int64_t base = t * kTile + (int64_t)w * (64 * kRadixIters) + lane;
    uint64_t k[kRadixIters];
    uint32_t v[kPacked ? 1 : kRadixIters];
#pragma unroll
    for (int it = 0; it < kRadixIters; it++) {
        const int64_t e = base + it * 64;
        k[it] = e < n ? kin[e] : 0ull;
        if (!kPacked) v[it] = e < n ? (vin ? vin[e] : (uint32_t)e) : 0u;
    }
    // counts of this wavefront (its own LDS row; leaders only, in step order)
    uint32_t place[kRadixIters];
#pragma unroll
    for (int it = 0; it < kRadixIters; it++) {
        const bool act = base + it * 64 < n;
        const uint32_t d = (uint32_t)(k[it] >> shift) & dmask;
        place[it] = step_place(d, D, act);
        if (act && (place[it] >> 16)) o[w][d] += (place[it] >> 8) & 0xffu;
    }
    __syncthreads();
    // digit starts inside the tile, then every wavefront's start per digit
    digit_starts<kPer>(o, nd, lstart, s_tot);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRadixIters; it++) {
        const bool act = base + it * 64 < n;
        const uint32_t d = (uint32_t)(k[it] >> shift) & dmask;
        const uint32_t start = act ? o[w][d] : 0u;
        if (act) {
            const uint32_t lp = start + (place[it] & 0xffu);
            sk[lp] = k[it];
            if (!kPacked) sv[lp] = v[it];
        }
        // LDS operations of one wavefront complete in order: every lane of the
        // group has read `start` before the leader's update lands
        if (act && (place[it] >> 16)) o[w][d] = start + ((place[it] >> 8) & 0xffu);
    }
    // lstart becomes the distance from a place in the tile to one in the output
    __syncthreads();
    for (int d = tid; d < nd; d += 256) lstart[d] = hscan[(int64_t)d * ntiles + t] - lstart[d];
    __syncthreads();
    const int64_t rem = n - t * kTile;
    const int cnt = rem < kTile ? (int)rem : (int)kTile;
    for (int lp = tid; lp < cnt; lp += 256) {
        const uint64_t key = sk[lp];
        const uint32_t d = (uint32_t)(key >> shift) & dmask;
        const uint32_t dst = lstart[d] + (uint32_t)lp;
        kout[dst] = key;
        if (!kPacked) vout[dst] = sv[lp];
    }
}

// Sorted slot s, key k (without index bits), original index o: the particle's
// two float4 records, its sub-cell and, when densities follow, its density
// record; and its cell once more on its own, for the kernels that only need
// that.
struct Sorted {
    float4 *__restrict__ spos, *__restrict__ sloc, *__restrict__ pq;
    uint16_t *__restrict__ ssub;
    uint32_t *__restrict__ scell;
};
__device__ __forceinline__ void place_particle(const float *__restrict__ pos, const Boxes &bx, int64_t s, uint64_t k,
                                               uint32_t o, const Sorted &to) {
    const uint32_t nsub = (uint32_t)bx.nsub_max;
    const uint32_t c = (uint32_t)(k / nsub);
    const uint32_t sub = (uint32_t)(k - (uint64_t)c * nsub);
    const Geo &g = bx.geo[box_of(bx, (uint32_t)s)];
    const float x = pos[3 * (int64_t)o + 0], y = pos[3 * (int64_t)o + 1], z = pos[3 * (int64_t)o + 2];
    to.spos[s] = make_float4(x, y, z, __uint_as_float(o));
    const uint32_t nc = (uint32_t)g.nc, lc = c - g.cell_base;
    const uint32_t cx = lc % nc, cy = (lc / nc) % nc, cz = lc / (nc * nc);
    const float xl = (float)(((double)x - (double)cx * g.cell) * g.inv_b);
    const float yl = (float)(((double)y - (double)cy * g.cell) * g.inv_b);
    const float zl = (float)(((double)z - (double)cz * g.cell) * g.inv_b);
    to.sloc[s] = make_float4(xl, yl, zl, __uint_as_float(c));
    if (to.pq) {
        // coordinates about the cell centre and minus their squared norm
        const float c0 = 0.5f * g.cellb;
        const float xc = xl - c0, yc = yl - c0, zc = zl - c0;
        to.pq[s] = make_float4(xc, yc, zc, -(xc * xc + yc * yc + zc * zc));
    }
    to.ssub[s] = (uint16_t)sub;
    to.scell[s] = c;
}

// pq's padding (read past a cell's end by the density kernel, never used).
__device__ __forceinline__ void place_padding(int64_t n, int64_t s, const Sorted &to) {
    if (to.pq && s < 32) to.pq[n + s] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

template <bool kPacked>
__global__ __launch_bounds__(kBlock) void k_bin_place(const float *__restrict__ pos, int64_t n, Boxes bx, int ib,
                                                      const uint64_t *__restrict__ key,
                                                      const uint32_t *__restrict__ idx, Sorted to) {
    const int64_t s = (int64_t)xcd_block() * blockDim.x + threadIdx.x;
    place_padding(n, s, to);
    if (s >= n) return;
    const uint64_t kw = key[s];
    place_particle(pos, bx, s, kPacked ? kw >> ib : kw,
                   kPacked ? (uint32_t)(kw & ((1ull << ib) - 1ull)) : idx[s], to);
}

// One stable pass of a workgroup over m words in memory, tile by tile, the
// digits' places running on from one tile to the next.
template <int NW = kRadixWaves, class Row>
__device__ __forceinline__ void big_bucket_pass(const uint64_t *src, uint64_t *dst, int64_t m, int sh, int D,
                                                uint32_t *run, Row o, uint32_t *s_tot) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, tid = threadIdx.x;
    const int nd = 1 << D;
    const uint32_t dmask = (uint32_t)(nd - 1);
    for (int d = tid; d < nd; d += 64 * NW) run[d] = 0u;
    __syncthreads();
    for (int64_t e = tid; e < m; e += 64 * NW) atomicAdd(&run[(uint32_t)(src[e] >> sh) & dmask], 1u);
    __syncthreads();
    const uint32_t first = block_scan_excl<NW>(tid < nd ? run[tid] : 0u, s_tot);
    __syncthreads();
    if (tid < nd) run[tid] = first;
    for (int64_t t0 = 0; t0 < m; t0 += 64 * NW * kRadixIters) {
        const int64_t e0 = t0 + w * (64 * kRadixIters) + lane;
        for (int d = lane; d < nd; d += 64) o[w][d] = 0u;
        uint64_t k[kRadixIters];
#pragma unroll
        for (int it = 0; it < kRadixIters; it++) k[it] = e0 + it * 64 < m ? src[e0 + it * 64] : 0ull;
        uint32_t place[kRadixIters];
#pragma unroll
        for (int it = 0; it < kRadixIters; it++) {
            const bool act = e0 + it * 64 < m;
            const uint32_t d = (uint32_t)(k[it] >> sh) & dmask;
            place[it] = step_place(d, D, act);
            if (act && (place[it] >> 16)) o[w][d] += (place[it] >> 8) & 0xffu;
        }
        __syncthreads();
        if (tid < nd) {
            uint32_t at = run[tid];
            for (int x = 0; x < NW; x++) {
                const uint32_t c = o[x][tid];
                o[x][tid] = at;
                at += c;
            }
            run[tid] = at;
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kRadixIters; it++) {
            const bool act = e0 + it * 64 < m;
            const uint32_t d = (uint32_t)(k[it] >> sh) & dmask;
            const uint32_t at = act ? o[w][d] : 0u;
            if (act) dst[at + (place[it] & 0xffu)] = k[it];
            if (act && (place[it] >> 16)) o[w][d] = at + ((place[it] >> 8) & 0xffu);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------- long buckets
// A bucket is a range of keys, part of a plane of cells, so a sheet of particles
// fills a few of them, and a workgroup per bucket is then the whole sort.  A
// bucket too long for LDS is therefore shared by several workgroups, each with a
// range of its keys: every one counts the bucket's particles in bins of
// consecutive keys, takes the bins that start in its share of the sorted order,
// gathers their particles in order and sorts them as a bucket of their own.
// Nobody waits for another workgroup.  (Half of the particles in one plane of
// cells, the whole binning: 5.0e5 particles 537 us with a workgroup per bucket,
// 139 with shares; 6.0e5 424 and 192; 2.0e6 609 and 292.)

// Share `part` of `parts` of the m particles counted in hist (PER bins per
// thread): the bins [lo, hi), the particles before them, and those in them.
struct Share {
    uint32_t lo, hi;
    int64_t first, cnt;
};
template <int PER, int NW>
__device__ __forceinline__ Share bin_share(const uint32_t *hist, int64_t m, int64_t part, int64_t parts,
                                           uint32_t *s_tot, uint32_t *s_sel) {
    const int64_t each = (m + parts - 1) / parts, from = part * each, to = from + each;
    const uint32_t bin0 = threadIdx.x * PER;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; q++) {
        c[q] = hist[bin0 + q];
        sum += c[q];
    }
    if (threadIdx.x < 2) {  // of a bound that no bin starts at or after
        s_sel[threadIdx.x] = 64 * NW * PER;
        s_sel[2 + threadIdx.x] = (uint32_t)m;
    }
    int64_t at = block_scan_excl<NW>(sum, s_tot);  // (with a barrier)
    int64_t prev = threadIdx.x > 0 ? at - (int64_t)hist[bin0 - 1] : -1;  // start of the bin before
#pragma unroll
    for (int q = 0; q < PER; q++) {
        if (prev < from && at >= from) {
            s_sel[0] = bin0 + q;
            s_sel[2] = (uint32_t)at;
        }
        if (prev < to && at >= to) {
            s_sel[1] = bin0 + q;
            s_sel[3] = (uint32_t)at;
        }
        prev = at;
        at += c[q];
    }
    __syncthreads();
    // the same words for all, in scalar registers: the workgroup branches on them
    // between barriers
    auto word = [&](int k) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)s_sel[k]); };
    const Share r{word(0), word(1), (int64_t)word(2), (int64_t)word(3) - (int64_t)word(2)};
    __syncthreads();  // hist and s_tot are free
    return r;
}

// Some of the elements [0, m) gathered in order: load(u, e) fetches element e as
// the lane's u-th of a round of kGather, take(u) tells whether it is one of them,
// and put(u, place, e) stores it.
constexpr int kGather = 4;
template <int NW, class Load, class Take, class Put>
__device__ __forceinline__ void gather_share(int64_t m, uint32_t *s_tot, Load load, Take take, Put put) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t run = 0;
    for (int64_t t0 = 0; t0 < m; t0 += 64 * NW * kGather) {
        const int64_t e0 = t0 + w * (64 * kGather) + lane;
#pragma unroll
        for (int u = 0; u < kGather; u++)
            if (e0 + u * 64 < m) load(u, e0 + u * 64);
        uint64_t mask[kGather];
        uint32_t mine = 0;
#pragma unroll
        for (int u = 0; u < kGather; u++) {
            mask[u] = __ballot(e0 + u * 64 < m && take(u));
            mine += (uint32_t)__popcll(mask[u]);
        }
        if (lane == 0) s_tot[w] = mine;
        __syncthreads();
        uint32_t at = run;
#pragma unroll
        for (int x = 0; x < NW; x++) {
            at += x < w ? s_tot[x] : 0u;
            run += s_tot[x];
        }
#pragma unroll
        for (int u = 0; u < kGather; u++) {
            if ((mask[u] >> lane) & 1ull) put(u, at + (uint32_t)__popcll(mask[u] & lanes_below(lane)), e0 + u * 64);
            at += (uint32_t)__popcll(mask[u]);
        }
        __syncthreads();
    }
}

// One bucket of the partition pass (the keys with the same bits above shift +
// bits), sorted by the bits [shift, shift + bits) with a stable radix sort of
// its own, then its particles' sorted records.  Bucket b holds the elements
// [start[b * stride], start[(b + 1) * stride]) (the whole input when start is
// null).  Up to kLocal elements stay in registers and LDS: each pass counts the
// digits of every wavefront's run of consecutive elements, places the elements
// in LDS in digit order and reads them back.  A longer bucket is shared by the
// workgroups past the buckets' own: one for every kShareStep-th element of the
// partitioned order, which exits unless that element lies in such a bucket (at
// least two do in each).  A share that is still too long (many particles in one
// bin) is sorted tile by tile in `work` (16 bytes per particle).
// On small inputs the passes are launch latency: four passes of count, two scan
// launches and scatter (and k_bin_place) took 92 us on the 64^3 box.
constexpr int kLocalIters = 16;
constexpr int kLocal = 256 * kLocalIters;
constexpr int kShareStep = 2048;
__global__ __launch_bounds__(256) void k_bucket_sort(const uint64_t *__restrict__ kin, uint64_t *work, int64_t n,
                                                     const uint32_t *__restrict__ start, int64_t stride,
                                                     int nbuckets, int shift, int bits,
                                                     const float *__restrict__ pos, Boxes bx, int ib, Sorted to) {
    constexpr int kPer = 8, kBinBits = 11;  // bins of a long bucket
    static_assert(256 * kPer == 1 << kBinBits, "bins of a long bucket");
    __shared__ uint32_t o[kRadixWaves][1 << kRadixMaxBits];
    __shared__ uint32_t lstart[1 << kRadixMaxBits], run[1 << kRadixMaxBits];
    __shared__ uint32_t s_tot[kRadixWaves], s_sel[4];
    __shared__ uint64_t sk[kLocal];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, tid = threadIdx.x;
    if (blockIdx.x == 0) place_padding(n, tid, to);
    const int passes = (bits + kRadixMaxBits - 1) / kRadixMaxBits;
    const int D = passes > 0 ? (bits + passes - 1) / passes : 0;
    const int nd = 1 << D;
    const uint32_t dmask = (uint32_t)(nd - 1);
    int64_t b0, m;  // the workgroup's elements: [b0, b0 + m) of the output
    uint64_t k[kLocalIters];
    if ((int)blockIdx.x < nbuckets) {
        b0 = start ? (int64_t)start[blockIdx.x * stride] : 0;
        m = (start ? (int64_t)start[(blockIdx.x + 1) * stride] : n) - b0;
        if (m <= 0 || m > kLocal) return;
        const int iters = (int)((m + 255) / 256), e0 = w * 64 * iters + lane;
#pragma unroll
        for (int it = 0; it < kLocalIters; it++)
            k[it] = it < iters && e0 + it * 64 < m ? kin[b0 + e0 + it * 64] : 0ull;
    } else {
        // the bucket of element p: its start is the last at or before p (256
        // starts probed at once, then those between two of them)
        const int64_t e = (int64_t)blockIdx.x - nbuckets, p = e * kShareStep;
        const int per = (nbuckets + 255) / 256;
        const int g = __syncthreads_count(tid * per < nbuckets && (int64_t)start[tid * per * stride] <= p) - 1;
        const int b = g * per - 1 +
                      __syncthreads_count(tid < per && g * per + tid < nbuckets &&
                                          (int64_t)start[(g * per + tid) * stride] <= p);
        b0 = start[b * stride];
        m = (int64_t)start[(b + 1) * stride] - b0;
        if (m <= kLocal) return;
        const int64_t e0 = (b0 + kShareStep - 1) / kShareStep, e1 = (b0 + m + kShareStep - 1) / kShareStep;
        // bins of the top bits of those to sort by
        const int bsh = shift + (bits > kBinBits ? bits - kBinBits : 0);
        auto bin = [&](uint64_t x) { return (uint32_t)((x & ((1ull << (shift + bits)) - 1ull)) >> bsh); };
        uint32_t *const hist = reinterpret_cast<uint32_t *>(sk);
        for (int q = tid; q < 256 * kPer; q += 256) hist[q] = 0u;
        __syncthreads();
        for (int64_t t = tid; t < m; t += 256 * kGather) {
            uint64_t x[kGather];
#pragma unroll
            for (int u = 0; u < kGather; u++) x[u] = t + u * 256 < m ? kin[b0 + t + u * 256] : 0ull;
#pragma unroll
            for (int u = 0; u < kGather; u++)
                if (t + u * 256 < m) atomicAdd(&hist[bin(x[u])], 1u);
        }
        __syncthreads();
        const Share sh = bin_share<kPer, kRadixWaves>(hist, m, e - e0, e1 - e0, s_tot, s_sel);
        if (sh.cnt <= 0) return;
        uint64_t *src = work + 2 * (b0 + sh.first), *dst = src + sh.cnt;
        uint64_t *const at = sh.cnt <= kLocal ? sk : src;
        uint64_t x[kGather];
        gather_share<kRadixWaves>(
            m, s_tot, [&](int u, int64_t i) { x[u] = kin[b0 + i]; },
            [&](int u) { return bin(x[u]) >= sh.lo && bin(x[u]) < sh.hi; },
            [&](int u, uint32_t place, int64_t) { at[place] = x[u]; });
        b0 += sh.first;
        m = sh.cnt;
        if (m > kLocal) {
            for (int q = 0; q < passes; q++) {
                big_bucket_pass(src, dst, m, shift + q * D, D, run, o, s_tot);
                uint64_t *const t = src;
                src = dst;
                dst = t;
            }
            for (int64_t s = tid; s < m; s += 256) {
                const uint64_t kw = src[s];
                place_particle(pos, bx, b0 + s, kw >> ib, (uint32_t)(kw & ((1ull << ib) - 1ull)), to);
            }
            return;
        }
        const int iters = (int)((m + 255) / 256), i0 = w * 64 * iters + lane;
#pragma unroll
        for (int it = 0; it < kLocalIters; it++) k[it] = it < iters && i0 + it * 64 < m ? sk[i0 + it * 64] : 0ull;
        __syncthreads();
    }
    const int iters = (int)((m + 255) / 256);  // elements per thread
    const int e0 = w * 64 * iters + lane;
    for (int p = 0; p < passes; p++) {
        const int sh = shift + p * D;
        for (int d = lane; d < nd; d += 64) o[w][d] = 0u;
        uint32_t place[kLocalIters];
#pragma unroll
        for (int it = 0; it < kLocalIters; it++) {
            place[it] = 0u;
            if (it < iters) {
                const bool act = e0 + it * 64 < m;
                const uint32_t d = (uint32_t)(k[it] >> sh) & dmask;
                place[it] = step_place(d, D, act);
                if (act && (place[it] >> 16)) o[w][d] += (place[it] >> 8) & 0xffu;
            }
        }
        __syncthreads();
        digit_starts<1>(o, nd, lstart, s_tot);
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kLocalIters; it++) {
            if (it < iters) {
                const bool act = e0 + it * 64 < m;
                const uint32_t d = (uint32_t)(k[it] >> sh) & dmask;
                const uint32_t at = act ? o[w][d] : 0u;
                if (act) sk[at + (place[it] & 0xffu)] = k[it];
                if (act && (place[it] >> 16)) o[w][d] = at + ((place[it] >> 8) & 0xffu);
            }
        }
        __syncthreads();
        if (p + 1 < passes) {
#pragma unroll
            for (int it = 0; it < kLocalIters; it++)
                if (it < iters && e0 + it * 64 < m) k[it] = sk[e0 + it * 64];
            __syncthreads();
        }
    }
    if (passes == 0) {
#pragma unroll
        for (int it = 0; it < kLocalIters; it++)
            if (it < iters && e0 + it * 64 < m) sk[e0 + it * 64] = k[it];
        __syncthreads();
    }
    for (int64_t s = tid; s < m; s += 256) {
        const uint64_t kw = sk[s];
        place_particle(pos, bx, b0 + s, kw >> ib, (uint32_t)(kw & ((1ull << ib) - 1ull)), to);
    }
}

// ------------------------------------------------- the sort that carries positions
// Two stable passes over digits of at most kRecBits bits, the low top bits and
// then the high ones, move records (x, y, z, index) instead of key words: the
// input positions are read in order twice and never gathered, where the gather
// of 12 bytes per particle took a 128-byte line each (460 us on the 256^3 box,
// 4.7 ms on the 512^3 one).  The key is computed again from the position
// wherever it is needed; the second digit travels beside the record.
constexpr int kRecBits = 9;

struct RecPlan {
    int low;     // key bits below the top ones, sorted within a bucket
    int dl, dh;  // bits of the first (low) and second (high) digit
};

// Positions of the elements e0, e0 + step, ... of this thread in input order,
// loaded together (past the end: the last one's).
struct TilePos {
    float x[kRadixIters], y[kRadixIters], z[kRadixIters];
};
__device__ __forceinline__ void tile_positions(const float *__restrict__ pos, int64_t n, int64_t e0, int step,
                                               TilePos &p) {
#pragma unroll
    for (int u = 0; u < kRadixIters; u++) {
        const int64_t i = e0 + (int64_t)u * step;
        const int64_t q = i < n ? i : n - 1;
        p.x[u] = pos[3 * q + 0];
        p.y[u] = pos[3 * q + 1];
        p.z[u] = pos[3 * q + 2];
    }
}

// f(constants of the box of input particle i): of the only box (g0, loaded once
// by the kernel), or through the box table.
template <bool kOne, class F>
__device__ __forceinline__ void with_box(const Boxes &bx, const Geo &g0, uint32_t i, F f) {
    if constexpr (kOne) f(g0);
    else per_box(bx, box_of(bx, i), f);
}

// The top key bits of the position of input particle i; *ok: it lies in its box.
template <bool kOne>
__device__ __forceinline__ uint32_t top_key(const Boxes &bx, const Geo &g0, uint32_t i, float x, float y, float z, int low, bool *ok) {
    uint32_t top = 0;
    bool in = true;
    with_box<kOne>(bx, g0, i, [&](const Geo &g) {
        in = inside(g, x, y, z);
        top = (uint32_t)(spot_of(g, bx.nsub_max, x, y, z).key >> low);
    });
    *ok = in;
    return top;
}

template <bool kOne>
__global__ __launch_bounds__(256) void k_rec_count(const float *__restrict__ pos, int64_t n, Boxes bx, RecPlan rp,
                                                   int64_t ntiles, uint32_t *__restrict__ hist,
                                                   int32_t *__restrict__ err) {
    __shared__ uint32_t h[1 << kRecBits];
    const int64_t t = xcd_block();
    const int nd = 1 << rp.dl;
    for (int d = threadIdx.x; d < nd; d += 256) h[d] = 0u;
    const Geo g0 = box_constants(bx, 0);
    TilePos p;
    tile_positions(pos, n, t * kTile + threadIdx.x, 256, p);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRadixIters; u++) {
        const int64_t i = t * kTile + threadIdx.x + u * 256;
        if (i < n) {
            bool ok;
            const uint32_t top = top_key<kOne>(bx, g0, (uint32_t)i, p.x[u], p.y[u], p.z[u], rp.low, &ok);
            if (!ok) flag_error(err, 1, box_of(bx, (uint32_t)i));
            atomicAdd(&h[top & (uint32_t)(nd - 1)], 1u);
        }
    }
    counts_out(h, nd, t, ntiles, hist);
}

// Counts of the second digit (in the order the first pass left).
__global__ __launch_bounds__(256) void k_rec_count2(const uint16_t *__restrict__ digit, int64_t n, int D,
                                                    int64_t ntiles, uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[1 << kRecBits];
    const int64_t t = xcd_block();
    const int nd = 1 << D;
    for (int d = threadIdx.x; d < nd; d += 256) h[d] = 0u;
    const int64_t base = t * kTile + threadIdx.x;
    uint16_t v[kRadixIters];
#pragma unroll
    for (int it = 0; it < kRadixIters; it++) v[it] = base + it * 256 < n ? digit[base + it * 256] : (uint16_t)0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRadixIters; it++)
        if (base + it * 256 < n) atomicAdd(&h[v[it]], 1u);
    counts_out(h, nd, t, ntiles, hist);
}

// Stable scatter of one tile's records by a digit.  kFirst: the records come
// from the input positions, by the first digit, with the second beside them;
// else from the first pass's records, by the second digit.
template <bool kFirst, bool kOne>
__global__ __launch_bounds__(256) void k_rec_scatter(const float *__restrict__ pos, const float4 *__restrict__ rin,
                                                     const uint16_t *__restrict__ din, int64_t n, Boxes bx,
                                                     RecPlan rp, int64_t ntiles,
                                                     const uint32_t *__restrict__ hscan, float4 *__restrict__ rout,
                                                     uint16_t *__restrict__ dout) {
    constexpr int kPer = (1 << kRecBits) / 256;
    __shared__ uint32_t o[kRadixWaves][1 << kRecBits];
    __shared__ uint32_t lstart[1 << kRecBits];
    __shared__ uint32_t s_tot[kRadixWaves];
    __shared__ float4 sr[kTile];
    __shared__ uint32_t sd[kTile];  // digit of this pass, and the second digit above it
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, tid = threadIdx.x;
    const int64_t t = xcd_block();
    const int D = kFirst ? rp.dl : rp.dh, nd = 1 << D;
    for (int d = lane; d < nd; d += 64) o[w][d] = 0u;
    const int64_t base = t * kTile + (int64_t)w * (64 * kRadixIters) + lane;
    TilePos p;
    uint32_t id[kRadixIters], dig[kRadixIters], place[kRadixIters];
    if (kFirst) {
        const Geo g0 = box_constants(bx, 0);
        tile_positions(pos, n, base, 64, p);
#pragma unroll
        for (int it = 0; it < kRadixIters; it++) {
            const int64_t e = base + it * 64;
            id[it] = (uint32_t)(e < n ? e : n - 1);
            bool ok;
            const uint32_t top = top_key<kOne>(bx, g0, id[it], p.x[it], p.y[it], p.z[it], rp.low, &ok);
            dig[it] = (top & (uint32_t)(nd - 1)) | ((top >> D) << 16);
        }
    } else {
#pragma unroll
        for (int it = 0; it < kRadixIters; it++) {
            const int64_t e = base + it * 64;
            const float4 r = rin[e < n ? e : n - 1];
            p.x[it] = r.x;
            p.y[it] = r.y;
            p.z[it] = r.z;
            id[it] = __float_as_uint(r.w);
            dig[it] = din[e < n ? e : n - 1];
        }
    }
#pragma unroll
    for (int it = 0; it < kRadixIters; it++) {
        const bool act = base + it * 64 < n;
        const uint32_t d = dig[it] & 0xffffu;
        place[it] = step_place(d, D, act);
        if (act && (place[it] >> 16)) o[w][d] += (place[it] >> 8) & 0xffu;
    }
    __syncthreads();
    digit_starts<kPer>(o, nd, lstart, s_tot);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRadixIters; it++) {
        const bool act = base + it * 64 < n;
        const uint32_t d = dig[it] & 0xffffu;
        const uint32_t start = act ? o[w][d] : 0u;
        if (act) {
            sr[start + (place[it] & 0xffu)] = make_float4(p.x[it], p.y[it], p.z[it], __uint_as_float(id[it]));
            sd[start + (place[it] & 0xffu)] = dig[it];
        }
        if (act && (place[it] >> 16)) o[w][d] = start + ((place[it] >> 8) & 0xffu);
    }
    __syncthreads();
    for (int d = tid; d < nd; d += 256) lstart[d] = hscan[(int64_t)d * ntiles + t] - lstart[d];
    __syncthreads();
    const int64_t rem = n - t * kTile;
    const int cnt = rem < kTile ? (int)rem : (int)kTile;
    for (int lp = tid; lp < cnt; lp += 256) {
        const uint32_t d = sd[lp];
        const uint32_t dst = lstart[d & 0xffffu] + (uint32_t)lp;
        rout[dst] = sr[lp];
        if (kFirst) dout[dst] = (uint16_t)(d >> 16);
    }
}

// First element of every bucket (high digit, low digit) after the second pass,
// and the total at the end: with p the first element of the low digit after
// the first pass, those of a high digit before p are the scanned count of p's
// tile and the ones of the tile before p.  One workgroup per low digit.
__global__ __launch_bounds__(256) void k_rec_starts(int64_t n, RecPlan rp, int64_t ntiles,
                                                    const uint32_t *__restrict__ first,
                                                    const uint32_t *__restrict__ hscan,
                                                    const uint16_t *__restrict__ digit,
                                                    uint32_t *__restrict__ starts) {
    __shared__ uint32_t h[1 << kRecBits];
    const int nh = 1 << rp.dh, nl = 1 << rp.dl;
    const int64_t p = first[blockIdx.x];
    const int64_t t = p < n ? p / kTile : ntiles - 1, t0 = t * kTile;
    for (int d = threadIdx.x; d < nh; d += 256) h[d] = 0u;
    __syncthreads();
    for (int64_t e = t0 + threadIdx.x; e < p; e += 256) atomicAdd(&h[digit[e]], 1u);
    __syncthreads();
    for (int d = threadIdx.x; d < nh; d += 256)
        starts[(int64_t)d * nl + blockIdx.x] = hscan[(int64_t)d * ntiles + t] + h[d];
    if (blockIdx.x == 0 && threadIdx.x == 0) starts[(int64_t)nh * nl] = (uint32_t)n;
}

// The first elements of the low digits after the first pass, kept from its
// scanned counts (the second pass's take their place), and after them the zero
// that the list of large buckets starts from.
__global__ __launch_bounds__(256) void k_rec_first(int nl, int64_t ntiles, const uint32_t *__restrict__ hscan,
                                                   uint32_t *__restrict__ first) {
    const int d = blockIdx.x * 256 + threadIdx.x;
    if (d <= nl) first[d] = d < nl ? hscan[(int64_t)d * ntiles] : 0u;
}

// The sorted records of slot s from the particle's record and its key (the low
// 32 bits: the sub-cell is what is left of it beyond the cell).
template <bool kOne>
__device__ __forceinline__ void place_record(const float4 &r, uint32_t key, const Boxes &bx, const Geo &g0, int64_t s,
                                             const Sorted &to) {
    with_box<kOne>(bx, g0, __float_as_uint(r.w), [&](const Geo &g) {
        const int cx = cell_coord(r.x, g), cy = cell_coord(r.y, g), cz = cell_coord(r.z, g);
        const uint32_t c =
            g.cell_base + ((uint32_t)cz * (uint32_t)g.nc + (uint32_t)cy) * (uint32_t)g.nc + (uint32_t)cx;
        to.spos[s] = r;
        const float xl = (float)(((double)r.x - (double)cx * g.cell) * g.inv_b);
        const float yl = (float)(((double)r.y - (double)cy * g.cell) * g.inv_b);
        const float zl = (float)(((double)r.z - (double)cz * g.cell) * g.inv_b);
        to.sloc[s] = make_float4(xl, yl, zl, __uint_as_float(c));
        if (to.pq) {
            // coordinates about the cell centre and minus their squared norm
            const float c0 = 0.5f * g.cellb;
            const float xc = xl - c0, yc = yl - c0, zc = zl - c0;
            to.pq[s] = make_float4(xc, yc, zc, -(xc * xc + yc * yc + zc * zc));
        }
        to.ssub[s] = (uint16_t)(key - c * (uint32_t)bx.nsub_max);
        to.scell[s] = c;
    });
}

// Buckets: their particles sorted by the low key bits (words of low bits and
// place in the bucket, in registers and LDS) and their sorted records written.
// A bucket is one workgroup's chain of dependent steps, so its length decides:
// 256 threads take buckets of up to 8 elements each (2048 particles) and list
// the longer ones (in `big`, pairs of bucket and share), which 1024 threads take
// with up to 16 each, one workgroup per listed share (a grid striding over the
// list).  A bucket beyond kRecMost particles is listed as several shares
// (rec_shares), found by bins of consecutive cells; a share that is still beyond
// kRecMost (a cell of so many) is sorted tile by tile in its part of `work` (16
// bytes per particle, as two arrays of 64-bit words).  (256 threads with 16
// elements and the tile sort beyond 4096 had 2.8 wavefronts per SIMD on average
// on the 256^3 box, most of the time a few long buckets: 563 us.)  The buckets are
// dealt to the XCDs in slices, since long ones lie together: 3.1M particles 82 ->
// 64 us, the 256^3 box 332 -> 279, the 512^3 box 2250 -> 1917 for 256 threads.
constexpr int kLowMost = 18;  // low key bits beside 14 bits of place
constexpr int kRecMost = 1 << 14;
// Shares of a bucket of m of all n particles: each reads the whole bucket twice,
// so as many as would run at once (256) if all buckets were like it, of at least a
// quarter of kRecMost, but of three quarters where that makes too many.  (Half of
// 1e7 particles in a plane of cells, buckets of 1.7e5: the binning 1.49 ms with
// quarters, 1.07 so; 1.11 by the radix sort when it came with a table over the
// grid.)
__device__ __forceinline__ int64_t rec_shares(int64_t m, int64_t n) {
    if (m <= kRecMost) return 1;
    const int64_t most = (m + kRecMost / 4 - 1) / (kRecMost / 4), least = (m + kRecMost / 4 * 3 - 1) / (kRecMost / 4 * 3);
    return min(min(max(256 * m / n, least), most), (int64_t)256);
}
template <int NW, int ITERS, bool kListed, bool kOne>
__global__ __launch_bounds__(64 * NW) void k_rec_bucket(const float4 *__restrict__ rec, int64_t n,
                                                        const uint32_t *__restrict__ starts, int low, Boxes bx,
                                                        uint64_t *work, uint32_t *__restrict__ big,
                                                        uint32_t *__restrict__ nbig, Sorted to) {
    constexpr int NT = 64 * NW, kMost = NT * ITERS, kPlace = 14;
    constexpr uint32_t kPlaces = (1u << kPlace) - 1u;
    static_assert(kMost <= 1 << kPlace && (!kListed || kMost == kRecMost), "14 bits of place");
    __shared__ uint32_t o[NW][1 << kRadixMaxBits];
    __shared__ uint32_t lstart[1 << kRadixMaxBits], run[kListed ? 1 << kRadixMaxBits : 1];
    __shared__ uint32_t s_tot[NW], s_sel[4];
    __shared__ uint32_t sk[kMost];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, tid = threadIdx.x;
    const int passes = (low + kRadixMaxBits - 1) / kRadixMaxBits;
    const int D = passes > 0 ? (low + passes - 1) / passes : 0;
    const int nd = 1 << D;
    const uint32_t dmask = (uint32_t)(nd - 1);
    const uint64_t lmask = (1ull << low) - 1ull;
    const Geo g0 = box_constants(bx, 0);
    if (!kListed && blockIdx.x == 0) place_padding(n, tid, to);
    const uint32_t nq = kListed ? *nbig : gridDim.x;
    for (uint32_t q = blockIdx.x; q < nq; q += gridDim.x) {
        const int64_t bucket = kListed ? big[2 * q] : xcd_tile_block(kXcdTile);
        const int64_t r0 = starts[bucket], rm = (int64_t)starts[bucket + 1] - r0;
        if (rm <= 0) return;  // only unlisted buckets, one per workgroup, are empty
        if (!kListed && rm > kMost) {
            const uint32_t parts = (uint32_t)rec_shares(rm, n);
            if (tid == 0) s_sel[0] = atomicAdd(nbig, parts);
            __syncthreads();
            const uint32_t at = s_sel[0];
            for (uint32_t p = tid; p < parts; p += NT) {
                big[2 * (at + p)] = (uint32_t)bucket;
                big[2 * (at + p) + 1] = p;
            }
            return;
        }
        auto low_key = [&](const float4 &r) -> uint32_t {
            uint32_t k = 0;
            with_box<kOne>(bx, g0, __float_as_uint(r.w), [&](const Geo &g) {
                k = (uint32_t)(spot_of(g, bx.nsub_max, r.x, r.y, r.z).key & lmask);
            });
            return k;
        };
        const uint32_t high = (uint32_t)((uint64_t)bucket << low);  // of the keys' low 32 bits
        int64_t b0 = r0, m = rm;  // the particles to sort: [b0, b0 + m) of the output
        const bool shared = kListed && rm > kMost;
        uint32_t *sidx = nullptr;  // a share's places in the bucket, by place in the share
        if constexpr (kListed) {
            if (shared) {
                // bins of consecutive cells (no sub-cells: an eighth of the key's arithmetic)
                constexpr int kPer = 4;
                constexpr uint32_t kBins = NT * kPer;
                const uint64_t key0 = (uint64_t)bucket << low;
                const uint32_t c0 = (uint32_t)(key0 / (uint64_t)bx.nsub_max);
                const uint32_t span = (uint32_t)((key0 + lmask) / (uint64_t)bx.nsub_max - c0);
                int bsh = 0;
                while (span >> bsh >= kBins) bsh++;
                auto bin = [&](const float4 &r) -> uint32_t {
                    uint32_t c = 0;
                    with_box<kOne>(bx, g0, __float_as_uint(r.w), [&](const Geo &g) {
                        const int cx = cell_coord(r.x, g), cy = cell_coord(r.y, g), cz = cell_coord(r.z, g);
                        c = g.cell_base + ((uint32_t)cz * (uint32_t)g.nc + (uint32_t)cy) * (uint32_t)g.nc +
                            (uint32_t)cx;
                    });
                    return (c - c0) >> bsh;
                };
                for (uint32_t d = tid; d < kBins; d += NT) sk[d] = 0u;
                __syncthreads();
                for (int64_t t = tid; t < rm; t += NT * kGather) {
                    float4 r[kGather];
#pragma unroll
                    for (int u = 0; u < kGather; u++) r[u] = rec[r0 + (t + u * NT < rm ? t + u * NT : 0)];
#pragma unroll
                    for (int u = 0; u < kGather; u++)
                        if (t + u * NT < rm) atomicAdd(&sk[bin(r[u])], 1u);
                }
                __syncthreads();
                const Share sh = bin_share<kPer, NW>(sk, rm, big[2 * q + 1], rec_shares(rm, n), s_tot, s_sel);
                if (sh.cnt <= 0) continue;
                b0 += sh.first;
                m = sh.cnt;
                uint64_t *src = work + 2 * b0, *dst = src + m;
                const bool fits = m <= kMost;
                sidx = reinterpret_cast<uint32_t *>(src);
                float4 r[kGather];
                gather_share<NW>(
                    rm, s_tot, [&](int u, int64_t i) { r[u] = rec[r0 + i]; },
                    [&](int u) {
                        const uint32_t d = bin(r[u]);
                        return d >= sh.lo && d < sh.hi;
                    },
                    [&](int u, uint32_t place, int64_t i) {
                        const uint32_t key = low_key(r[u]);
                        if (fits) {
                            sk[place] = (key << kPlace) | place;
                            sidx[place] = (uint32_t)i;
                        } else {
                            src[place] = ((uint64_t)key << 32) | (uint64_t)i;
                        }
                    });
                if (!fits) {
                    for (int p = 0; p < passes; p++) {
                        big_bucket_pass<NW>(src, dst, m, 32 + p * D, D, run, o, s_tot);
                        uint64_t *const t = src;
                        src = dst;
                        dst = t;
                    }
                    for (int64_t s = tid; s < m; s += NT)
                        place_record<kOne>(rec[r0 + (int64_t)(src[s] & 0xffffffffull)],
                                           high + (uint32_t)(src[s] >> 32), bx, g0, b0 + s, to);
                    __syncthreads();  // LDS is free for the next listed share
                    continue;
                }
            }
        }
        const int iters = (int)((m + NT - 1) / NT);  // elements per thread
        const int e0 = w * 64 * iters + lane;
        uint32_t k[ITERS];
        if (!shared) {
            // keys to LDS in order (two records in flight), then each thread's
            // elements to registers: a rolled loop keeps the key arithmetic out
            // of the unrolled passes
            for (int it = 0; it < iters; it += 2) {
                const int ea = e0 + it * 64, eb = ea + 64;
                const bool ina = ea < m, inb = it + 1 < iters && eb < m;
                const float4 ra = rec[r0 + (ina ? ea : 0)], rb = rec[r0 + (inb ? eb : 0)];
                const uint32_t ka = low_key(ra), kb = low_key(rb);
                if (ina) sk[ea] = (ka << kPlace) | (uint32_t)ea;
                if (inb) sk[eb] = (kb << kPlace) | (uint32_t)eb;
            }
        }
#pragma unroll
        for (int it = 0; it < ITERS; it++) k[it] = it < iters && e0 + it * 64 < m ? sk[e0 + it * 64] : 0u;
        __syncthreads();
        for (int p = 0; p < passes; p++) {
            const int sh = kPlace + p * D;
            for (int d = lane; d < nd; d += 64) o[w][d] = 0u;
            uint32_t place[ITERS];
#pragma unroll
            for (int it = 0; it < ITERS; it++) {
                place[it] = 0u;
                if (it < iters) {
                    const bool act = e0 + it * 64 < m;
                    const uint32_t d = (k[it] >> sh) & dmask;
                    place[it] = step_place(d, D, act);
                    if (act && (place[it] >> 16)) o[w][d] += (place[it] >> 8) & 0xffu;
                }
            }
            __syncthreads();
            digit_starts<1, NW>(o, nd, lstart, s_tot);
            __syncthreads();
#pragma unroll
            for (int it = 0; it < ITERS; it++) {
                if (it < iters) {
                    const bool act = e0 + it * 64 < m;
                    const uint32_t d = (k[it] >> sh) & dmask;
                    const uint32_t at = act ? o[w][d] : 0u;
                    if (act) sk[at + (place[it] & 0xffu)] = k[it];
                    if (act && (place[it] >> 16)) o[w][d] = at + ((place[it] >> 8) & 0xffu);
                }
            }
            __syncthreads();
            if (p + 1 < passes) {
#pragma unroll
                for (int it = 0; it < ITERS; it++)
                    if (it < iters && e0 + it * 64 < m) k[it] = sk[e0 + it * 64];
                __syncthreads();
            }
        }
        auto record = [&](uint32_t word) {
            const uint32_t at = word & kPlaces;
            return rec[r0 + (shared ? sidx[at] : at)];
        };
        for (int s = tid; s < m; s += 2 * NT) {
            const bool two = s + NT < m;
            const uint32_t wa = sk[s], wb = two ? sk[s + NT] : wa;
            const float4 ra = record(wa), rb = record(wb);
            place_record<kOne>(ra, high + (wa >> kPlace), bx, g0, b0 + s, to);
            if (two) place_record<kOne>(rb, high + (wb >> kPlace), bx, g0, b0 + s + NT, to);
        }
        if (!kListed) return;
        __syncthreads();  // LDS is free for the next listed share
    }
}

// First sorted particle of the cell cc that holds particle s0 - 1, by a wavefront:
// the 64 particles before that one, then steps back of doubling length, then
// the interval between two of them cut 65-fold.
__device__ __forceinline__ int64_t cell_start(const uint32_t *__restrict__ scell, int64_t s0, uint32_t cc) {
    const int lane = threadIdx.x & 63;
    int64_t hi = s0 - 1;  // in the cell
    auto in = [&](int64_t p) { return p >= 0 && scell[p] == cc; };
    uint64_t m = ~__ballot(in(hi - 1 - lane));
    if (m) return hi - __builtin_ctzll(m);
    hi -= 64;
    // lane 63 would step back 2^69 particles: all past the first 33 miss
    const int64_t back = (int64_t)64 << min(lane, 33);
    m = ~__ballot(in(hi - back));
    const int f = __builtin_ctzll(m);  // the first step out of the cell
    int64_t lo = hi - ((int64_t)64 << f);
    if (f > 0) hi -= (int64_t)64 << (f - 1);
    if (lo < -1) lo = -1;
    // lo is not in the cell, hi is
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + 64) / 65;
        const int64_t p = lo + step * (lane + 1);
        const uint64_t q = __ballot(p >= hi || in(p));
        const int k = q ? __builtin_ctzll(q) : 64;  // the first probe in the cell
        const int64_t top = lo + step * (k + 1);
        lo += step * k;
        if (k < 64 && top < hi) hi = top;
    }
    return hi;
}

constexpr int kFineTile = 1024;
constexpr int64_t kFineTilesMost = (int64_t)1 << 22;  // 4096 tiles

// Marks of the sorted particles: head of a dense chunk, head of a dense cell,
// sparse, head of a cell.  A wavefront takes 64 consecutive particles at a time
// and finds the bounds of their cells from the cell ids of neighbouring
// particles (cell changes are found by ballot); only where a cell starts before
// the wavefront's particles is its start searched for, and where one ends after
// them one more id tells whether it is dense.  The marks are kept as the ballots
// (a word per kind and particle, and its scan, moved 70 bytes per particle and
// took eleven launches), and a workgroup's kTile particles leave the four counts
// for the scan of the lists.  The words of the cell index are zeroed for the
// next kernel (zero: nzero of them).
template <int kTile>
__global__ __launch_bounds__(kBlock) void k_bin_marks(int64_t n, const uint32_t *__restrict__ scell, Marks marks,
                                                      uint32_t *__restrict__ sums, int64_t tiles,
                                                      uint2 *__restrict__ zero, int64_t nzero) {
    __shared__ uint32_t s_cnt[kBlock / 64][4];
    constexpr int kSteps = kTile / kBlock, kIlp = 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int64_t z = (int64_t)blockIdx.x * kBlock + threadIdx.x; z < nzero; z += (int64_t)gridDim.x * kBlock)
        zero[z] = make_uint2(0u, 0u);
    const int64_t t = xcd_block();
    uint32_t nc = 0, nd = 0, ns = 0, nh = 0;
    for (int k0 = 0; k0 < kSteps; k0 += kIlp) {
        // each step's cells, and those beyond its two ends (lane 0: the slot
        // before it, lane 63: the one after), all loaded together
        uint32_t c[kIlp], ce[kIlp];
#pragma unroll
        for (int u = 0; u < kIlp; u++) {
            const int64_t s0 = t * kTile + ((k0 + u) * (kBlock / 64) + w) * 64, i = s0 + lane;
            const int64_t e = lane == 0 ? s0 - 1 : (lane == 63 ? s0 + 64 : -1);
            c[u] = i < n ? scell[i] : 0xffffffffu;
            ce[u] = e >= 0 && e < n ? scell[e] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kIlp; u++) {
            const int64_t s0 = t * kTile + ((k0 + u) * (kBlock / 64) + w) * 64, i = s0 + lane;
            if (s0 >= n) break;
            const bool act = i < n;
            uint32_t cprev = __shfl_up(c[u], 1, 64), cnext = __shfl_down(c[u], 1, 64);
            if (lane == 0) cprev = s0 > 0 ? ce[u] : ~c[u];
            if (lane == 63) cnext = s0 + 64 < n ? ce[u] : ~c[u];
            if (i + 1 == n) cnext = ~c[u];
            const uint64_t heads = __ballot(act && c[u] != cprev);
            const uint64_t tails = __ballot(act && c[u] != cnext);
            const uint64_t le = lane == 63 ? ~0ull : ((1ull << (lane + 1)) - 1ull);
            const uint64_t h = heads & le, tl = tails & ~(le >> 1);  // heads at or below, tails at or above
            // the start of the cell, for the first cell possibly before s0
            int64_t before = s0;
            if (!(heads & 1ull)) before = cell_start(scell, s0, lane_get(c[u], 0));
            const int64_t a = h ? s0 + 63 - __clzll((long long)h) : before;
            bool dense;
            if (tl)
                dense = s0 + __ffsll((unsigned long long)tl) - a >= kDenseMin;
            else  // holds the particle after the wavefront's too
                dense = a + kDenseMin - 1 <= s0 + 64 ||
                        (a + kDenseMin - 1 < n && scell[a + kDenseMin - 1] == c[u]);
            dense = dense && act;
            const bool head = dense && ((i - a) & 63) == 0, first = dense && i == a;
            const uint64_t mc = __ballot(head), md = __ballot(first), ms = __ballot(act && !dense);
            if (lane == 0) {
                marks.chunk[s0 >> 6] = mc;
                marks.dcell[s0 >> 6] = md;
                marks.sparse[s0 >> 6] = ms;
                marks.head[s0 >> 6] = heads;
            }
            nc += (uint32_t)__popcll(mc);
            nd += (uint32_t)__popcll(md);
            ns += (uint32_t)__popcll(ms);
            nh += (uint32_t)__popcll(heads);
        }
    }
    if (lane == 0) {
        s_cnt[w][0] = nc;
        s_cnt[w][1] = nd;
        s_cnt[w][2] = ns;
        s_cnt[w][3] = nh;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        uint32_t v = 0;
        for (int x = 0; x < kBlock / 64; x++) v += s_cnt[x][threadIdx.x];
        sums[threadIdx.x * tiles + t] = v;
    }
}

// The lists of the marked particles, a workgroup per kTile particles: dense
// chunks, dense cells (their cell and its number, and the map back) and sparse
// particles, with the zeros that the sparse particles' dense-neighbour sums
// start from (dfx may be null), and the cell index: the cells that start in the
// tile are gathered in LDS in order, and the first of each word writes it.  Only
// a word shared with a neighbouring tile takes an atomic.  The last workgroup
// leaves the totals in the counters.
template <int kTile>
__global__ __launch_bounds__(kBlock) void k_bin_lists(int64_t n, Marks marks, const uint32_t *__restrict__ sums,
                                                      int64_t tiles, bool scanned,
                                                      const uint32_t *__restrict__ scell,
                                                      int32_t *__restrict__ chunks,
                                                      uint32_t *__restrict__ dcells,
                                                      uint32_t *__restrict__ dord,
                                                      int32_t *__restrict__ sparse, Cells cells,
                                                      uint64_t *__restrict__ dfx,
                                                      int32_t *__restrict__ counters,
                                                      uint32_t *__restrict__ zero, int nzero) {
    constexpr int kWords = kTile / 64, kKinds = 4, kIlp = 4;
    static_assert(kWords <= 64 && kBlock / 64 == kKinds, "one lane per word, one wavefront per kind");
    static_assert(kWords % (kKinds * kIlp) == 0, "whole rounds");
    __shared__ uint64_t s_mark[kKinds][kWords];
    __shared__ uint32_t s_at[kKinds][kWords];
    __shared__ uint32_t s_cell[kTile];
    __shared__ uint32_t s_heads, s_first;
    __shared__ bool s_shared;  // the tile's first cell shares its word with the cell before it
    const int64_t t = xcd_block();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // the counts of the next stage's segmented list start here
    if (blockIdx.x == 0)
        for (int q = threadIdx.x; q < nzero; q += kBlock) zero[q] = 0u;
    // wavefront w: the words of kind w and the marked particles before each
    {
        uint32_t off = 0;
        if (t > 0 && scanned) off = sums[w * tiles + t];
        else if (t > 0) {
            for (int64_t q = lane; q < t; q += 4 * 64) {
#pragma unroll
                for (int u = 0; u < 4; u++) off += q + 64 * u < t ? sums[w * tiles + q + 64 * u] : 0u;
            }
            for (int d = 32; d >= 1; d >>= 1) off += __shfl_xor(off, d, 64);
        }
        const int64_t word = t * kWords + lane;
        const bool in = lane < kWords && word * 64 < n;
        const uint64_t *p = w == 0 ? marks.chunk : (w == 1 ? marks.dcell : (w == 2 ? marks.sparse : marks.head));
        const uint64_t m = in ? p[word] : 0ull;
        const uint32_t cnt = (uint32_t)__popcll(m), incl = wave_incl_scan(cnt);
        const uint32_t at = off + incl - cnt;
        if (lane < kWords) {
            s_mark[w][lane] = m;
            s_at[w][lane] = at;
        }
        if (w == 1 && in) marks.dbefore[word] = at;
        if (w == 2 && in) marks.before[word] = at;
        if (w == 3 && lane == 63) {
            s_heads = incl;
            s_first = off;
        }
        if (t == tiles - 1 && lane == 63) {
            if (w == 3) cells.start[at + cnt] = (uint32_t)n;
            else counters[w == 0 ? kCntChunks : (w == 1 ? kCntDcells : kCntSparse)] = (int32_t)(at + cnt);
        }
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
    const uint32_t ofirst = s_first;  // number of the tile's first cell
    for (int k0 = w; k0 < kWords; k0 += kKinds * kIlp) {
        uint32_t c[kIlp];
#pragma unroll
        for (int u = 0; u < kIlp; u++) {
            const int64_t i = (t * kWords + k0 + kKinds * u) * 64 + lane;
            c[u] = i < n ? scell[i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kIlp; u++) {
            const int k = k0 + kKinds * u;
            const int64_t i = (t * kWords + k) * 64 + lane;
            const uint64_t mc = s_mark[0][k], md = s_mark[1][k], ms = s_mark[2][k], mh = s_mark[3][k];
            if ((mc >> lane) & 1ull) chunks[s_at[0][k] + (uint32_t)__popcll(mc & below)] = (int32_t)i;
            if ((ms >> lane) & 1ull) {
                const uint32_t at = s_at[2][k] + (uint32_t)__popcll(ms & below);
                sparse[at] = (int32_t)i;
                if (dfx) dfx[at] = 0ull;
            }
            if ((mh >> lane) & 1ull) {
                const uint32_t o = s_at[3][k] + (uint32_t)__popcll(mh & below), q = o - ofirst;
                cells.start[o] = (uint32_t)i;
                s_cell[q] = c[u];
                if (q == 0u) s_shared = i > 0 && scell[i - 1] / kOccCells == c[u] / kOccCells;
                if ((md >> lane) & 1ull) {
                    const uint32_t d = s_at[1][k] + (uint32_t)__popcll(md & below);
                    dcells[d] = c[u];
                    dord[d] = o;
                    cells.dmap[o] = d;
                }
            }
        }
    }
    __syncthreads();
    const uint32_t heads = s_heads;
    for (uint32_t q = threadIdx.x; q < heads; q += kBlock) {
        const uint32_t word = s_cell[q] / kOccCells;
        if (q > 0u && s_cell[q - 1u] / kOccCells == word) continue;
        uint32_t bits = 0, r = q;
        for (; r < heads && s_cell[r] / kOccCells == word; r++) bits |= 1u << (s_cell[r] % kOccCells);
        uint2 *const e = cells.occ + word;
        const bool joins = q == 0u && s_shared;
        if (joins || r == heads) {
            atomicOr(&e->x, bits);
            if (!joins) e->y = ofirst + q;
        } else {
            *e = make_uint2(bits, ofirst + q);
        }
    }
}

// Sub-cell table of one dense cell d, by one wavefront: entry s is the first
// particle of the cell whose sub-cell is s or later (an empty sub-cell gets
// the start of the next non-empty one; entry nsub is the cell end).  The
// cell's particles are sorted by sub-cell, so particle j writes the entries
// after its predecessor's sub-cell up to its own, and the entries after the
// last particle's sub-cell get the cell end; every entry is written once.
__device__ __forceinline__ void sub_table_cell(int64_t d, const Boxes &bx, const uint32_t *__restrict__ dord,
                                               const uint32_t *__restrict__ start,
                                               const uint16_t *__restrict__ ssub,
                                               uint32_t *__restrict__ subtab) {
    const int lane = threadIdx.x & 63;
    const uint32_t o = (uint32_t)__builtin_amdgcn_readfirstlane(dord[d]);
    const uint32_t a = (uint32_t)__builtin_amdgcn_readfirstlane(start[o]);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane(start[o + 1]);
    const int nsub = __builtin_amdgcn_readfirstlane(bx.geo[box_of(bx, a)].nsub);
    uint32_t *t = subtab + d * (bx.nsub_max + 1);
    for (uint32_t j0 = a; j0 < b; j0 += 64) {
        const uint32_t j = j0 + (uint32_t)lane;
        if (j < b) {
            const int cur = ssub[j];
            const int prev = j > a ? (int)ssub[j - 1] : -1;
            for (int s2 = prev + 1; s2 <= cur; s2++) t[s2] = j;
            if (j + 1 == b)
                for (int s2 = cur + 1; s2 <= nsub; s2++) t[s2] = b;
        }
    }
}

// The sub-cell tables of all dense cells, one wavefront per cell over a grid
// that strides the cells; the cell count *ndc_p is read on the device.
__global__ __launch_bounds__(kBlock) void k_sub_table(const uint32_t *__restrict__ ndc_p, Boxes bx,
                                                      const uint32_t *__restrict__ dord,
                                                      const uint32_t *__restrict__ start,
                                                      const uint16_t *__restrict__ ssub,
                                                      uint32_t *__restrict__ subtab) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t ndc = *ndc_p;
    const int64_t stride = (int64_t)gridDim.x * (kBlock / 64);
    for (int64_t d = (int64_t)blockIdx.x * (kBlock / 64) + wave; d < ndc; d += stride)
        sub_table_cell(d, bx, dord, start, ssub, subtab);
}

}  // namespace

int bit_width(uint64_t x) {
    int b = 0;
    while (b < 64 && (x >> b)) b++;
    return b;
}

// Particles up to which the sort is one partition pass over (key, index) words:
// up to 1024 buckets of 512 particles on average.  One bucket is then the
// longest chain: with 1300 on average (1.3e6 particles) the largest buckets
// passed kLocal and the bucket sort took 140 us instead of 33 us on 2.6e5.
constexpr int64_t kPartitionMost = (int64_t)1 << 19;

// Top bits of the partition pass: buckets of 256 to 512 particles on average.
int partition_bits(int64_t n) {
    const int top = bit_width((uint64_t)((n - 1) / 256));
    return top < kPartBits ? top : kPartBits;
}

// Sort plan: key bits; index bits when packed (0 = separate payload), and top
// bits of the buckets of the partition pass (-1: none); the digits of the sort
// that carries positions (dl < 0: none); the passes of D bits of the radix sort.
struct SortPlan {
    int bits, ib, top;
    RecPlan rec;
    int passes, D;
};

SortPlan sort_plan(int64_t n, int64_t ncell, int nsub_max) {
    const uint64_t nkeys = (uint64_t)ncell * (uint64_t)nsub_max;
    SortPlan r;
    r.bits = bit_width(nkeys - 1);
    if (r.bits < 1) r.bits = 1;
    r.passes = (r.bits + kRadixMaxBits - 1) / kRadixMaxBits;
    r.D = (r.bits + r.passes - 1) / r.passes;
    int ib = bit_width((uint64_t)(n > 1 ? n - 1 : 1));
    r.ib = ib + r.bits <= 64 ? ib : 0;
    // HF_RADIX_PAYLOAD=1 forces the radix sort with a separate payload (used by
    // tests; it is otherwise taken only when key and index need more than 64
    // bits)
    const char *force = getenv("HF_RADIX_PAYLOAD");
    const bool radix = force && force[0] == '1';
    if (radix) r.ib = 0;
    r.top = -1;
    r.rec = RecPlan{0, -1, -1};
    if (radix) return r;
    if (r.ib > 0 && n <= kPartitionMost) {
        r.top = partition_bits(n);
        if (r.top > r.bits) r.top = r.bits;
        return r;
    }
    // the records' second buffer (Work::rec2) lies over the sub-cell tables, 16
    // bytes an entry, which hold an entry per particle from 7 sub-cells on;
    // buckets of 300 to 1000 particles on average, so many that the low bits fit
    // beside the place in the bucket
    int top = bit_width((uint64_t)((n - 1) / 1024));
    if (top < r.bits - kLowMost) top = r.bits - kLowMost;
    if (top > 2 * kRecBits) top = 2 * kRecBits;
    if (top > r.bits) top = r.bits;
    // So this sort reaches keys of 36 bits, 18 top and 18 low ones: a 512^3 box at
    // the defaults has just that many; a larger one, or more than 27 sub-cells a
    // cell there, takes the radix sort below, and so does a grid of far more cells
    // than particles, whose buckets would hold a few each.
    if (sub_entries(n, nsub_max) >= n && top >= 2 && r.bits - top <= kLowMost && (n >> top) >= 128) {
        r.rec.low = r.bits - top;
        r.rec.dl = top / 2;
        r.rec.dh = top - r.rec.dl;
    }
    return r;
}

int64_t radix_hist_len(int64_t n) {
    // the widest digit of a sort of n particles, and of every radix sort of up to
    // n keys
    const int64_t ntiles = (n + kTile - 1) / kTile;
    const int first = n > kPartitionMost ? kRecBits : (n > 0 ? partition_bits(n) : 0);
    return ((int64_t)1 << (first > kRadixMaxBits ? first : kRadixMaxBits)) * (ntiles > 0 ? ntiles : 1) + 1;
}

int64_t bin_tiles(int64_t n) { return n <= kFineTilesMost ? (n + kFineTile - 1) / kFineTile : scan_tiles(n); }

uint64_t *radix_sort_keys(uint64_t *a, uint64_t *b, int64_t n, int lo, int bits, Work &w, hipStream_t s) {
    if (n <= 1 || bits <= 0) return a;
    const int passes = (bits + kRadixMaxBits - 1) / kRadixMaxBits;
    const int D = (bits + passes - 1) / passes;
    const int64_t ntiles = (n + kTile - 1) / kTile;
    const int64_t hl = ((int64_t)1 << D) * ntiles;
    uint64_t *cur = a, *nxt = b;
    for (int p = 0; p < passes; p++) {
        const int shift = lo + p * D;
        hipLaunchKernelGGL(k_radix_count, dim3((unsigned)ntiles), dim3(256), 0, s, cur, n, shift, D, ntiles,
                           w.rhist);
        scan_u32(w.rhist, w.rscan, hl, w.scan_tmp, s);
        hipLaunchKernelGGL((k_radix_scatter<true, kRadixMaxBits>), dim3((unsigned)ntiles), dim3(256), 0, s, cur,
                           nullptr, n, shift, D, ntiles, w.rscan, nxt, nullptr);
        uint64_t *t = cur;
        cur = nxt;
        nxt = t;
    }
    return cur;
}

void launch_bin(const float *pos, int64_t n, int64_t ncell, const Boxes &bx, Work &w, hipStream_t s) {
    const SortPlan r = sort_plan(n, ncell, bx.nsub_max);
    const bool packed = r.ib > 0;
    const int64_t ntiles = (n + kTile - 1) / kTile;
    const dim3 tiles((unsigned)ntiles);
    const Sorted to{w.spos, w.sloc, w.pq, w.ssub, w.scell};
    if (r.top >= 0) {
        const int low = r.bits - r.top, shift = r.ib + low;
        hipLaunchKernelGGL(k_bin_key, tiles, dim3(256), 0, s, pos, n, bx, r.ib, w.rkey[0], shift, r.top, ntiles,
                           w.rhist, w.err);
        const uint32_t *start = nullptr;
        int cur = 0;
        if (r.top > 0) {
            scan_u32(w.rhist, w.rscan, ((int64_t)1 << r.top) * ntiles, w.scan_tmp, s);
            hipLaunchKernelGGL((k_radix_scatter<true, kPartBits>), tiles, dim3(256), 0, s, w.rkey[0], nullptr, n,
                               shift, r.top, ntiles, w.rscan, w.rkey[1], nullptr);
            start = w.rscan;
            cur = 1;
        }
        // long buckets: a workgroup for every kShareStep particles, and their
        // tile sorts in the scratch run (16 bytes per particle)
        const int64_t shares = n > kLocal ? (n + kShareStep - 1) / kShareStep : 0;
        hipLaunchKernelGGL(k_bucket_sort, dim3((1u << r.top) + (unsigned)shares), dim3(256), 0, s, w.rkey[cur],
                           reinterpret_cast<uint64_t *>(w.tmp_a), n, start, ntiles, 1 << r.top, r.ib, low, pos, bx,
                           r.ib, to);
    } else if (r.rec.dl >= 0) {
        // first pass into the radix key block (16 bytes per particle), second
        // over the sub-cell tables, which are written after the binning; the
        // second digits lie in the sub-cell indices' array and the buckets'
        // starts in the radix payload (both free until the buckets are sorted,
        // which read neither after writing them)
        float4 *ra = reinterpret_cast<float4 *>(w.rkey[0]), *rb = w.rec2;
        const int nl = 1 << r.rec.dl, nh = 1 << r.rec.dh;
        const bool one = bx.nbox == 1;
        hipLaunchKernelGGL(one ? k_rec_count<true> : k_rec_count<false>, tiles, dim3(256), 0, s, pos, n, bx, r.rec,
                           ntiles, w.rhist, w.err);
        scan_u32(w.rhist, w.rscan, (int64_t)nl * ntiles, w.scan_tmp, s);
        hipLaunchKernelGGL((one ? k_rec_scatter<true, true> : k_rec_scatter<true, false>), tiles, dim3(256), 0, s, pos,
                           nullptr, nullptr, n, bx, r.rec, ntiles, w.rscan, ra, w.ssub);
        hipLaunchKernelGGL(k_rec_first, dim3((unsigned)(nl + 1 + 255) / 256), dim3(256), 0, s, nl, ntiles, w.rscan,
                           w.rval[1]);
        hipLaunchKernelGGL(k_rec_count2, tiles, dim3(256), 0, s, w.ssub, n, r.rec.dh, ntiles, w.rhist);
        scan_u32(w.rhist, w.rscan, (int64_t)nh * ntiles, w.scan_tmp, s);
        hipLaunchKernelGGL((k_rec_scatter<false, true>), tiles, dim3(256), 0, s, nullptr, ra, w.ssub, n, bx, r.rec,
                           ntiles, w.rscan, rb, nullptr);
        hipLaunchKernelGGL(k_rec_starts, dim3((unsigned)nl), dim3(256), 0, s, n, r.rec, ntiles, w.rval[1], w.rscan,
                           w.ssub, w.rval[0]);
        // the list of long buckets' shares and its count after those first elements
        uint32_t *nbig = w.rval[1] + nl, *big = nbig + 1;
        hipLaunchKernelGGL((one ? k_rec_bucket<4, 8, false, true> : k_rec_bucket<4, 8, false, false>),
                           dim3((unsigned)(nl * nh)), dim3(256), 0, s, rb, n, w.rval[0], r.rec.low, bx, w.rkey[0], big,
                           nbig, to);
        const int64_t most = n / 2048 + 1;  // more than 2048 particles each
        hipLaunchKernelGGL((one ? k_rec_bucket<16, 16, true, true> : k_rec_bucket<16, 16, true, false>),
                           dim3((unsigned)(most < 512 ? most : 512)), dim3(1024), 0, s, rb, n, w.rval[0], r.rec.low,
                           bx, w.rkey[0], big, nbig, to);
    } else {
        hipLaunchKernelGGL(k_bin_key, tiles, dim3(256), 0, s, pos, n, bx, r.ib, w.rkey[0], r.ib, r.D, ntiles, w.rhist,
                           w.err);
        const int64_t hl = ((int64_t)1 << r.D) * ntiles;
        int cur = 0;
        for (int p = 0; p < r.passes; p++) {
            const int shift = r.ib + p * r.D;
            if (p > 0)
                hipLaunchKernelGGL(k_radix_count, tiles, dim3(256), 0, s, w.rkey[cur], n, shift, r.D, ntiles,
                                   w.rhist);
            scan_u32(w.rhist, w.rscan, hl, w.scan_tmp, s);
            if (packed)
                hipLaunchKernelGGL((k_radix_scatter<true, kRadixMaxBits>), tiles, dim3(256), 0, s, w.rkey[cur],
                                   nullptr, n, shift, r.D, ntiles, w.rscan, w.rkey[cur ^ 1], nullptr);
            else
                hipLaunchKernelGGL((k_radix_scatter<false, kRadixMaxBits>), tiles, dim3(256), 0, s, w.rkey[cur],
                                   p == 0 ? nullptr : w.rval[cur], n, shift, r.D, ntiles, w.rscan,
                                   w.rkey[cur ^ 1], w.rval[cur ^ 1]);
            cur ^= 1;
        }
        if (packed)
            hipLaunchKernelGGL(k_bin_place<true>, dim3(blocks(n)), dim3(kBlock), 0, s, pos, n, bx, r.ib, w.rkey[cur],
                               nullptr, to);
        else
            hipLaunchKernelGGL(k_bin_place<false>, dim3(blocks(n)), dim3(kBlock), 0, s, pos, n, bx, 0, w.rkey[cur],
                               w.rval[cur], to);
    }
    // tiles of 4096 particles, of 1024 where those would leave most of the chip
    // idle and a workgroup's rounds be the time (20 000 particles: the two
    // kernels took 14 and 17 us, 5 and 8 with the smaller tiles)
    const bool fine = n <= kFineTilesMost;
    const int64_t lt = bin_tiles(n);
    // the index words are zeroed by the marks' workgroups, by a launch of their
    // own when there are too many for them (a nearly empty grid)
    const int64_t words = occ_words(ncell);
    const bool apart = words > 128 * kBlock * lt;
    if (apart) fill_u32(reinterpret_cast<uint32_t *>(w.cells.occ), 0u, 2 * words, s);
    hipLaunchKernelGGL(fine ? k_bin_marks<kFineTile> : k_bin_marks<kScanTile>, dim3((unsigned)lt), dim3(kBlock), 0, s, n,
                       w.scell, w.marks, w.scan_tmp, lt, w.cells.occ, apart ? 0 : words);
    const bool scanned = scan_sums(w.scan_tmp, lt, lt, 4, s);
    // the dense cells' numbers in the radix sort's payload (free by now)
    hipLaunchKernelGGL(fine ? k_bin_lists<kFineTile> : k_bin_lists<kScanTile>, dim3((unsigned)lt), dim3(kBlock), 0, s, n,
                       w.marks, w.scan_tmp, lt, scanned, w.scell, w.chunks, w.dcells, w.rval[0], w.sparse, w.cells,
                       w.pq ? w.rkey[0] : nullptr, w.counters, w.rhist, (int)(seg_list(n, w).nseg * kSegStride));
}

void launch_subtab(int64_t n, const uint32_t *ndc_p, const Boxes &bx, Work &w, hipStream_t s) {
    if (n <= 0) return;
    // the count is read on the device; a dense cell holds at least kDenseMin
    // particles, and a grid of at most 16384 workgroups strides over the cells
    const int64_t ub = n / kDenseMin + 1;
    int64_t blocks = (ub + kBlock / 64 - 1) / (kBlock / 64);
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_sub_table, dim3((unsigned)blocks), dim3(kBlock), 0, s, ndc_p, bx, w.rval[0],
                       w.cells.start, w.ssub, w.subtab);
}

}  // namespace hf
