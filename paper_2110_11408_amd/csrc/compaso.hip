// CompaSO L1 inside every L0 group (Sec. 2.2.2) and the output cut.
//
// The paper's per-group loop is sequential (find a nucleus, assign, mark
// ineligible, repeat).  It decomposes exactly into data-parallel stages because
//   - the peak condition and the nucleation floor depend only on the densities
//     (steps 2 and 4), so the candidate set is fixed before the loop;
//   - R_L1 of a nucleus uses ALL particles of the L0 group and is independent of
//     earlier assignments (steps 1-2);
//   - eligibility depends only on earlier nuclei and their R (step 1);
//   - a particle's reassignment depends only on its current halo (step 3).
// Hence: candidates are found in parallel; R is computed for all of them in
// parallel; a wavefront per group walks its candidates in descending density and
// rejects those inside alpha R of an accepted nucleus; finally every particle
// folds over its group's accepted halos in creation order.
//
// R without sorting (Sec. 2.3.3: the enclosed mass at sorted position k is k,
// R_L1 is where the enclosed density first drops below Delta_L1).  With
// T(e) = K^2 e^3 for a squared distance e (R^3 = i/K), the sorted definition
// "first k >= 1 whose k-th smallest T exceeds k^2" is equivalent to
// "first k >= 1 with C(k) <= k", where C(k) counts particles with T <= k^2.
// C is the prefix sum of a histogram over integer buckets
// ceil(sqrt(T)) (computed exactly with integer-square comparisons), so each
// candidate costs a pass or two over the group and a prefix scan.
#include "hf_internal.h"
#include "scan_tile.h"

namespace hf {

namespace {

inline dim3 grid(int64_t n) { return dim3((unsigned)((n + kBlock - 1) / kBlock)); }

__device__ __forceinline__ int32_t ldi(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void sti(int32_t *p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------ segmentation

// The members of every group are counted by the kernels that write the group
// keys (gcnt[key], zero before).  Two prefix sums over the keys, of the counts
// and of their non-zero ones, give every group its start and its ordinal.
__global__ __launch_bounds__(kBlock) void k_seg_sums(int64_t n, const uint32_t *__restrict__ gcnt,
                                                     uint32_t *__restrict__ msum, uint32_t *__restrict__ gsum,
                                                     uint64_t *clock) {
    stamp(clock);
    uint32_t m = 0, g = 0;
    tile_each(gcnt, (int64_t)blockIdx.x * kScanTile, n, [&](uint32_t c) {
        m += c;
        g += c != 0u ? 1u : 0u;
    });
    m = block_sum(m);
    g = block_sum(g);
    if (threadIdx.x == 0) {
        msum[blockIdx.x] = m;
        gsum[blockIdx.x] = g;
    }
}

// Totals of two runs of tile sums (one workgroup): members, groups.
__global__ __launch_bounds__(kBlock) void k_seg_totals(int64_t tiles, const uint32_t *__restrict__ msum,
                                                       const uint32_t *__restrict__ gsum,
                                                       int32_t *__restrict__ counters) {
    uint32_t m = 0, g = 0;
    for (int64_t t = threadIdx.x; t < tiles; t += kBlock) {
        m += msum[t];
        g += gsum[t];
    }
    m = block_sum(m);
    g = block_sum(g);
    if (threadIdx.x == 0) {
        counters[kCntMembers] = (int32_t)m;
        counters[kCntGroups] = (int32_t)g;
    }
}

// The prefixes of a tile of keys, stored for the keys of groups only: the
// group's start and ordinal by key, and by ordinal its start, size, label and
// the zeros its later counts start from.  (Whole prefix arrays and a fill per
// count array, with a kernel of their own for the per-group values, moved 32
// bytes per particle more and cost six more launches.)  Also zeroed here: the
// table-row bits (n / 32 + 1 words) and the words of `clear`.
__global__ __launch_bounds__(kBlock) void k_seg_offsets(int64_t n, const uint32_t *__restrict__ gcnt,
                                                        const uint32_t *__restrict__ msum,
                                                        const uint32_t *__restrict__ gsum, bool scanned,
                                                        uint32_t *__restrict__ goff, uint32_t *__restrict__ gidx,
                                                        int32_t *__restrict__ g_start,
                                                        int32_t *__restrict__ g_size,
                                                        int32_t *__restrict__ g_label,
                                                        uint32_t *__restrict__ gccnt,
                                                        uint32_t *__restrict__ gcfill,
                                                        int32_t *__restrict__ g_nh,
                                                        int32_t *__restrict__ gflag,
                                                        uint32_t *__restrict__ tflag, SegClear clear,
                                                        int32_t *__restrict__ counters) {
    __shared__ uint32_t buf[kScanLds];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    const int64_t word = (int64_t)blockIdx.x * (kScanTile / 32) + threadIdx.x;
    if (threadIdx.x <= kScanTile / 32 && word <= (n >> 5)) tflag[word] = 0u;
    if (blockIdx.x == 0)
        for (int k = 0; k < SegClear::kRuns; k++)
            for (int t = threadIdx.x; t < clear.len[k]; t += kBlock) clear.p[k][t] = 0u;
    uint32_t v[kScanItems];
    tile_load(gcnt, base, n, buf, v, [](uint32_t x) { return x; });
    uint32_t m = 0, g = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        m += v[k];
        g += v[k] != 0u ? 1u : 0u;
    }
    uint32_t mt, gt;
    uint32_t moff = block_excl_scan(m, &mt), goffs = block_excl_scan(g, &gt);
    const uint32_t m0 = blockIdx.x > 0 ? tile_offset(msum, blockIdx.x, scanned) : 0u;
    const uint32_t g0 = blockIdx.x > 0 ? tile_offset(gsum, blockIdx.x, scanned) : 0u;
    moff += m0;
    goffs += g0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        if (!v[k]) continue;
        const int64_t key = base + (int64_t)threadIdx.x * kScanItems + k;
        goff[key] = moff;
        gidx[key] = goffs;
        g_start[goffs] = (int32_t)moff;
        g_size[goffs] = (int32_t)v[k];
        g_label[goffs] = (int32_t)key + 1;
        gccnt[goffs] = 0u;
        gcfill[goffs] = 0u;
        g_nh[goffs] = 0;
        gflag[goffs] = 0;
        moff += v[k];
        goffs++;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        counters[kCntMembers] = (int32_t)(m0 + mt);
        counters[kCntGroups] = (int32_t)(g0 + gt);
    }
}

// Members into group order: each run of equal keys among consecutive lanes
// takes a slice of its group by counting the group's count down (the order of
// members inside a group is not used).
__global__ __launch_bounds__(kBlock) void k_seg_scatter(int64_t n, const int32_t *__restrict__ gkey,
                                                        const uint32_t *__restrict__ goff,
                                                        const uint32_t *__restrict__ gidx,
                                                        uint32_t *__restrict__ gcnt,
                                                        int32_t *__restrict__ mem,
                                                        int32_t *__restrict__ gid_of) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int k = i < n ? gkey[i] : -1;
    const WaveRun r = wave_run(k);
    uint32_t base = 0;
    if (k >= 0 && r.rank == 0) base = atomicSub(&gcnt[k], (uint32_t)r.len) - (uint32_t)r.len;
    base = __shfl(base, r.head, 64);
    if (i >= n) return;
    if (k < 0) {
        gid_of[i] = -1;
        return;
    }
    mem[goff[k] + base + (uint32_t)r.rank] = (int32_t)i;
    gid_of[i] = (int32_t)gidx[k];
}

// ------------------------------------------------------- group extent
// Every distance is a minimum image, which stands for the distance inside an
// L0 group only while the group spans less than half the box along each axis.
// A group whose extent reaches L/2 makes the call fail (HF_ERR_INVALID) rather
// than return labels computed with the wrong images.  The extent is measured
// from the group's first member r: with o_q the minimum-image offset of member
// q from r along an axis, extent = max o - min o.  Offsets below L/4 in every
// axis bound it below L/2, so a first pass flags the groups with a member at
// L/4 or more and the exact extent is taken for those only.

// Minimum-image offset b - a along one axis (the canonical fold).
__device__ __forceinline__ double mi_off(float a, float b, double L, double half) {
    double d = (double)b - (double)a;
    if (d > half) d -= L; else if (d < -half) d += L;
    return d;
}

__global__ __launch_bounds__(kBlock) void k_extent_far(const int32_t *__restrict__ members_p, Boxes bx, const int32_t *__restrict__ mem,
                                                       const int32_t *__restrict__ gid_of,
                                                       const int32_t *__restrict__ g_start,
                                                       const float4 *__restrict__ spos,
                                                       int32_t *__restrict__ gflag,
                                                       int32_t *__restrict__ farlist,
                                                       uint32_t *__restrict__ nfar) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)*members_p) return;
    const int i = mem[t];
    const Geo &g = bx.geo[box_of(bx, (uint32_t)i)];
    const int gi = gid_of[i];
    const float4 pr = spos[mem[g_start[gi]]];
    const float4 pi = spos[i];
    const double q = 0.25 * g.L;
    const bool far = fabs(mi_off(pr.x, pi.x, g.L, g.half)) >= q || fabs(mi_off(pr.y, pi.y, g.L, g.half)) >= q ||
                     fabs(mi_off(pr.z, pi.z, g.L, g.half)) >= q;
    if (far && atomicCAS(&gflag[gi], 0, 1) == 0) farlist[atomicAdd(nfar, 1u)] = gi;
}

// The exact extent of the flagged groups, one workgroup per group (grid-stride
// over the list, its length read on the device).
__global__ __launch_bounds__(kBlock) void k_extent_span(const uint32_t *__restrict__ nfar_p, Boxes bx,
                                                        const int32_t *__restrict__ farlist,
                                                        const int32_t *__restrict__ g_start,
                                                        const int32_t *__restrict__ g_size,
                                                        const int32_t *__restrict__ mem,
                                                        const float4 *__restrict__ spos,
                                                        int32_t *__restrict__ err) {
    __shared__ double s_lo[3][kBlock / 64], s_hi[3][kBlock / 64];
    const uint32_t nfar = *nfar_p;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (uint32_t f = blockIdx.x; f < nfar; f += gridDim.x) {
        const int gi = farlist[f];
        const int64_t start = g_start[gi], m = g_size[gi];
        const int box = __builtin_amdgcn_readfirstlane(box_of(bx, (uint32_t)mem[start]));
        const Geo &g = bx.geo[box];
        const float4 pr = spos[mem[start]];
        double lo[3] = {0.0, 0.0, 0.0}, hi[3] = {0.0, 0.0, 0.0};
        for (int64_t t = threadIdx.x; t < m; t += blockDim.x) {
            const float4 pq = spos[mem[start + t]];
            const double o[3] = {mi_off(pr.x, pq.x, g.L, g.half), mi_off(pr.y, pq.y, g.L, g.half),
                                 mi_off(pr.z, pq.z, g.L, g.half)};
#pragma unroll
            for (int a = 0; a < 3; a++) {
                lo[a] = fmin(lo[a], o[a]);
                hi[a] = fmax(hi[a], o[a]);
            }
        }
#pragma unroll
        for (int a = 0; a < 3; a++) {
            for (int d = 32; d >= 1; d >>= 1) {
                lo[a] = fmin(lo[a], __shfl_xor(lo[a], d, 64));
                hi[a] = fmax(hi[a], __shfl_xor(hi[a], d, 64));
            }
            if (lane == 0) {
                s_lo[a][wid] = lo[a];
                s_hi[a][wid] = hi[a];
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            bool wide = false;
            for (int a = 0; a < 3; a++) {
                double l = s_lo[a][0], h = s_hi[a][0];
                for (int w = 1; w < kBlock / 64; w++) {
                    l = fmin(l, s_lo[a][w]);
                    h = fmax(h, s_hi[a][w]);
                }
                wide = wide || h - l >= g.half;
            }
            if (wide) flag_error(err, 8, box);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------ acceptance and R
// Smallest integer k >= 0 with T <= k^2 (both sides as the FP64 expressions
// T and ii(k)); m when T > ii(m - 1) (beyond every k the search inspects).
__device__ __forceinline__ int64_t bucket_of(double T, int64_t m) {
    if (!(T > 0.0)) return 0;
    if (m <= 1 || T > ii(m - 1)) return m;
    // the loops below reach the exact k from any start in [0, m - 1]: the
    // start only sets their length, so it comes from the FP32 square root
    // (T < 2^62 here; within a few units of k below 2^23, one or two steps),
    // not from the much longer FP64 one
    int64_t k = (int64_t)ceilf(__builtin_amdgcn_sqrtf((float)T));
    if (k > m - 1) k = m - 1;
    if (k < 0) k = 0;
    while (k > 0 && T <= ii(k - 1)) k--;
    while (T > ii(k)) k++;
    return k;
}

constexpr int kHistMid = 2048;    // histogram buckets of a medium group, counted in LDS (8 KB)
constexpr int kHistBig = 36864;   // histogram buckets of a large group counted in LDS (144 KB)
constexpr int kScanIpt = 16;      // buckets per thread per scan step

// Block-wide exclusive scan of one value per thread (NT threads).
template <int NT>
__device__ __forceinline__ uint32_t block_excl(uint32_t v, uint32_t *s_red, uint32_t *total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t inc = v;
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t t = __shfl_up(inc, d, 64);
        if (lane >= d) inc += t;
    }
    if (lane == 63) s_red[wid] = inc;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
    for (int w = 0; w < NT / 64; w++) {
        if (w < wid) pre += s_red[w];
        tot += s_red[w];
    }
    __syncthreads();
    *total = tot;
    return pre + inc - v;
}

template <int NT>
__device__ __forceinline__ int block_min(int v, int *s_min) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int d = 32; d >= 1; d >>= 1) v = min(v, __shfl_xor(v, d, 64));
    if (lane == 0) s_min[wid] = v;
    __syncthreads();
    int best = s_min[0];
    for (int w = 1; w < NT / 64; w++) best = min(best, s_min[w]);
    __syncthreads();
    return best;
}

// Candidates (their places in cand_sorted) of groups that are not small: each
// group's densest from the front of the list, the others from its back (the
// list of the late ones has those at its front, and rests null).
struct AcceptItems {
    int32_t *list;
    uint32_t *firsts, *rests, cap;
};

constexpr int kWaveHist = 1024;   // groups of one candidate below this size run one per wavefront

// Groups with candidates (all boxes, largest first), one wavefront at a time
// each: a persistent grid of W wavefronts in which wavefront w takes groups
// w, w + W, w + 2W, ... of the list (its length read on the device), so that
// every wavefront gets one group of each size tier.  (A shared counter that
// every wavefront increments per group serialises on its one address: tens of
// thousands of groups cost more in atomics than in work.)  Groups of fewer
// than kWaveHist particles with one candidate, most of all groups, are settled
// here: the candidate is accepted, and its enclosed count found from a histogram
// in the wavefront's LDS with wave-level scans, so that many small groups run on
// a CU at once.  The candidates of the other groups go to the item lists of the
// medium groups (fewer than mid_most particles) or the large ones, for
// k_accept_eval (route_all: every group, when R is searched by radial bins).
// (With groups of up to 64 candidates walked here, the longest walk was the
// time: 17 us for 20 000 particles, 11 without.)
__global__ __launch_bounds__(kBlock) void k_accept_small(const uint32_t *__restrict__ ngc_p, bool route_all, int mid_most,
                                                         Boxes bx,
                                                         const int32_t *__restrict__ glist,
                                                         const int32_t *__restrict__ g_start,
                                                         const int32_t *__restrict__ g_size,
                                                         const uint32_t *__restrict__ gcoff,
                                                         const int32_t *__restrict__ cand_sorted,
                                                         const int32_t *__restrict__ mem,
                                                         const float4 *__restrict__ spos,
                                                         int32_t *__restrict__ h_nuc,
                                                         int32_t *__restrict__ h_ienc,
                                                         int32_t *__restrict__ h_gid,
                                                         int32_t *__restrict__ g_nh,
                                                         AcceptItems mid, AcceptItems big, AcceptItems late,
                                                         int late_most, int32_t *__restrict__ enc,
                                                         uint64_t *clock) {
#pragma clang fp contract(off)
    stamp(clock);
    __shared__ uint32_t s_hist[kBlock / 64][kWaveHist];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const uint32_t ngc = __builtin_amdgcn_readfirstlane(*ngc_p);
    const uint32_t nw = gridDim.x * (kBlock / 64);
    uint32_t *hist = s_hist[wave];
    for (uint32_t q = blockIdx.x * (kBlock / 64) + (uint32_t)wave; q < ngc; q += nw) {
        const int gi = glist[q];
        const int64_t start = g_start[gi];
        const int64_t m = g_size[gi];
        const Geo &g = bx.geo[__builtin_amdgcn_readfirstlane(box_of(bx, (uint32_t)mem[start]))];
        const uint32_t cs = gcoff[gi], ce = gcoff[gi + 1];
        if (route_all || m + 1 > kWaveHist || ce - cs > 1u) {
            const AcceptItems &to = m + 1 <= mid_most ? mid : big;
            const bool wait = m > late_most;
            uint32_t at = 0;
            if (lane == 0) {
                to.list[atomicAdd(to.firsts, 1u)] = (int32_t)cs;
                enc[cs] = -1;  // not known yet
                if (ce - cs > 1u) at = atomicAdd(wait ? late.firsts : to.rests, ce - cs - 1u);
            }
            at = lane_get(at, 0);
            for (uint32_t k = lane; k < ce - cs - 1u; k += 64) {
                const int32_t item = (int32_t)(cs + 1u + k);
                if (wait) late.list[at + k] = item;
                else to.list[to.cap - 1u - (at + k)] = item;
            }
            continue;
        }
        const int c = cand_sorted[cs];
        const float4 pc = spos[c];
        // bucket histogram over all m particles of the group
        for (int64_t k = lane; k <= m; k += 64) hist[k] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        // four members per lane and round of loads
        for (int64_t t0 = lane; t0 < m; t0 += 4 * 64) {
            int32_t id[4];
            float4 pm[4];
#pragma unroll
            for (int u = 0; u < 4; u++) id[u] = t0 + 64 * u < m ? mem[start + t0 + 64 * u] : c;
#pragma unroll
            for (int u = 0; u < 4; u++) pm[u] = spos[id[u]];
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (t0 + 64 * u < m) atomicAdd(&hist[bucket_of(g.K2 * e3(d2_exact(pc, pm[u], g.L, g.half)), m)], 1u);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        // first k in [1, m-1] with C(k) <= k, C(k) = sum of buckets 0..k;
        // lane L covers buckets 16L .. 16L + 15 (m < 1024)
        uint32_t v[16];
        uint32_t sum = 0;
#pragma unroll
        for (int u = 0; u < 16; u++) {
            const int64_t k = (int64_t)lane * 16 + u;
            v[u] = k < m ? hist[k] : 0u;
            sum += v[u];
        }
        uint32_t C = wave_incl_scan(sum) - sum;
        int hit = -1;
#pragma unroll
        for (int u = 0; u < 16; u++) {
            const int64_t k = (int64_t)lane * 16 + u;
            C += v[u];
            if (hit < 0 && k >= 1 && k < m && (int64_t)C <= k) hit = (int)k;
        }
        const uint64_t hm = __ballot(hit >= 0);
        const int64_t found = hm ? (int64_t)lane_get(hit, __ffsll((unsigned long long)hm) - 1) : m;
        if (lane == 0) {
            h_nuc[cs] = c;
            h_ienc[cs] = (int32_t)found;
            h_gid[cs] = gi;
            g_nh[gi] = 1;
        }
        __builtin_amdgcn_wave_barrier();  // the histogram is free for the next group
    }
}

// Squared outer edge of radial bin j of width w: ((j + 1) w)^2; bin j holds
// the squared distances e with edge(j - 1) <= e < edge(j).
__device__ __forceinline__ double rbin_edge2(int j, double w) {
    const double r = (double)(j + 1) * w;
    return r * r;
}

// The bin of e (the bin width is such that every minimum-image distance lies
// inside the last edge).
__device__ __forceinline__ int rbin_of(double e, double w) {
    int j = (int)(sqrt(e) / w);
    if (j > kRadBins - 1) j = kRadBins - 1;
    while (j > 0 && e < rbin_edge2(j - 1, w)) j--;
    while (j < kRadBins - 1 && !(e < rbin_edge2(j, w))) j++;
    return j;
}

// f(e) for the squared distance e of every member of the group to pc, the
// members spread over the workgroup (UB per thread and round, their loads
// issued together).
template <int NT, class F>
__device__ __forceinline__ void for_members(int64_t m, int64_t start, const int32_t *__restrict__ mem,
                                            const float4 *__restrict__ spos, const float4 &pc, const Geo &g,
                                            F f) {
    constexpr int UB = NT >= 1024 ? 4 : 8;
    for (int64_t t0 = threadIdx.x; t0 < m; t0 += UB * NT) {
        int32_t id[UB];
#pragma unroll
        for (int u = 0; u < UB; u++) {
            const int64_t t = t0 + (int64_t)u * NT;
            id[u] = t < m ? mem[start + t] : -1;
        }
        float4 pm[UB];
#pragma unroll
        for (int u = 0; u < UB; u++) pm[u] = id[u] >= 0 ? spos[id[u]] : pc;
#pragma unroll
        for (int u = 0; u < UB; u++)
            if (id[u] >= 0) f(d2_exact(pc, pm[u], g.L, g.half));
    }
}

// First t in [w0, w1) with C(t) <= t and 1 <= base + t <= m - 1, where
// C(t) = run + hist[0] + ... + hist[t - w0]; -1 when there is none (run then
// includes the whole window).
template <int NT>
__device__ __forceinline__ int64_t first_crossing(const uint32_t *s_hist, int64_t w0, int64_t w1, int64_t base,
                                                  int64_t m, uint32_t &run, uint32_t *s_red, int *s_min) {
    constexpr int SI = NT >= 1024 ? kScanIpt / 2 : kScanIpt;
    for (int64_t b0 = w0; b0 < w1; b0 += (int64_t)NT * SI) {
        const int64_t k0 = b0 + (int64_t)threadIdx.x * SI;
        uint32_t v[SI];
        uint32_t sum = 0;
#pragma unroll
        for (int u = 0; u < SI; u++) {
            const int64_t k = k0 + u;
            v[u] = k < w1 ? s_hist[k - w0] : 0u;
            sum += v[u];
        }
        uint32_t tot;
        uint32_t C = run + block_excl<NT>(sum, s_red, &tot);
        int hit = 0x7fffffff;
#pragma unroll
        for (int u = 0; u < SI; u++) {
            const int64_t k = k0 + u;
            C += v[u];
            if (hit == 0x7fffffff && k < w1 && base + k >= 1 && base + k < m && (int64_t)C <= k)
                hit = (int)(k - b0);
        }
        const int best = block_min<NT>(hit, s_min);
        run += tot;
        if (best != 0x7fffffff) return b0 + best;
    }
    return -1;
}

// First coarse bucket j < nj, of the 2^sh buckets from w0 + (j << sh) on, in which
// a crossing can lie: C before it is at most its last bucket (C only grows).
// run: C before w0, on return C before the bucket found.
template <int NT>
__device__ __forceinline__ int64_t first_possible(const uint32_t *s_hist, int64_t w0, int64_t nj, int sh,
                                                  uint32_t &run, uint32_t *s_red, int *s_min, uint32_t *s_c) {
    constexpr int SI = NT >= 1024 ? kScanIpt / 2 : kScanIpt;
    for (int64_t b0 = 0; b0 < nj; b0 += (int64_t)NT * SI) {
        const int64_t k0 = b0 + (int64_t)threadIdx.x * SI;
        uint32_t v[SI];
        uint32_t sum = 0;
#pragma unroll
        for (int u = 0; u < SI; u++) {
            v[u] = k0 + u < nj ? s_hist[k0 + u] : 0u;
            sum += v[u];
        }
        uint32_t tot;
        uint32_t C = run + block_excl<NT>(sum, s_red, &tot), Chit = 0;
        int hit = 0x7fffffff;
#pragma unroll
        for (int u = 0; u < SI; u++) {
            const int64_t k = k0 + u;
            if (hit == 0x7fffffff && k < nj && (int64_t)C <= w0 + ((k + 1) << sh) - 1) {
                hit = (int)(k - b0);
                Chit = C;
            }
            C += v[u];
        }
        const int best = block_min<NT>(hit, s_min);
        if (best != 0x7fffffff) {
            if (hit == best) *s_c = Chit;
            __syncthreads();
            run = *s_c;
            __syncthreads();
            return b0 + best;
        }
        run += tot;
    }
    return -1;
}

// The enclosed count i of every listed candidate, one workgroup at a time each.
// A candidate is accepted unless it lies inside alpha R of a nucleus accepted
// before it; i depends on the group and the candidate only.  Nearly every
// candidate is accepted (28 072 of 28 141 on the 256^3 box), so i is found for
// all of them at once instead of one after the other in the group's walk
// (k_accept_walk), whose chain was the time of the stage (5.7 ms on the 512^3 box,
// 289 us on the 256^3 one and 138 us on 1.3e6 particles at their labels; 2.9 ms,
// 170 us and 59 us now).  The groups'
// densest candidates come first; a candidate that lies inside alpha R of that
// one, if its i is known by then, is left out (its i is never asked for).  In
// large groups (accept_late) the others are a list and a launch of their own, so
// that it is.
//   BINS = false: i from the bucket histogram of all particles of the group, in
//                 LDS; with more buckets than fit (HL), half of it holds the
//                 first ones and the other half the rest in coarse ones, which
//                 tell from where on the buckets are looked at next (mostly one
//                 such step: few coarse buckets have C before them as low as
//                 their numbers, but the very first ones always do, so they
//                 must not be coarse: a group of 500 000 members took 8.0 ms in
//                 windows from the first bucket on, 1.17 so);
//   BINS = true:  by the radial bins of Sec. 2.3.4.  Counts of the members per
//                 radial bin (width g.rbin, in LDS) give C_j, the members
//                 inside bin j's inner edge.  A bin whose C_j members, placed
//                 at its outer edge, still meet the threshold
//                 (K^2 edge^3 <= C_j^2) holds no crossing: every member in it
//                 is inside that edge at a sorted position >= C_j.  The first
//                 bin that is not passed over is searched with the bucket
//                 histogram of its own members (positions C_j .. C_j + c_j - 1
//                 of the sorted order: the crossing is the first t with
//                 #{bin members with bucket <= C_j + t} <= t), HL of them at a
//                 time, and the search moves outwards while a bin holds no
//                 crossing.
template <int NT, int HL, bool BINS>
__global__ __launch_bounds__(NT) void k_accept_eval(AcceptItems items, Boxes bx,
                                                    const int32_t *__restrict__ gid_of,
                                                    const int32_t *__restrict__ g_start,
                                                    const int32_t *__restrict__ g_size,
                                                    const uint32_t *__restrict__ gcoff,
                                                    const int32_t *__restrict__ cand_sorted,
                                                    const int32_t *__restrict__ mem,
                                                    const float4 *__restrict__ spos,
                                                    int32_t *enc,
                                                    int32_t *__restrict__ h_nuc,
                                                    int32_t *__restrict__ h_ienc,
                                                    int32_t *__restrict__ h_gid,
                                                    int32_t *__restrict__ g_nh) {
#pragma clang fp contract(off)
    __shared__ uint32_t s_hist[HL];
    __shared__ uint32_t s_rb[BINS ? kRadBins : 1];
    __shared__ uint32_t s_red[NT / 64], s_c;
    __shared__ int s_min[NT / 64];
    const int tid = threadIdx.x;
    const uint32_t firsts = *items.firsts, count = firsts + (items.rests ? *items.rests : 0u);
    for (uint32_t q = blockIdx.x; q < count; q += gridDim.x) {
        const uint32_t cr = (uint32_t)items.list[q < firsts ? q : items.cap - 1u - (q - firsts)];
        const int c = cand_sorted[cr];
        const int gi = gid_of[c];
        const int64_t start = g_start[gi];
        const int64_t m = g_size[gi];
        const uint32_t cs = gcoff[gi], ce = gcoff[gi + 1];
        const Geo &g = bx.geo[__builtin_amdgcn_readfirstlane(box_of(bx, (uint32_t)c))];
        const float4 pc = spos[c];
        if (cr != cs) {
            // one answer for the workgroup: another one may write it meanwhile.
            // Scalar, so that the workgroup leaves for its next item as one.
            if (tid == 0) s_c = (uint32_t)ldi(enc + cs);
            __syncthreads();
            const int32_t i0 = __builtin_amdgcn_readfirstlane((int32_t)s_c);
            __syncthreads();
            const bool inside = i0 >= 0 && g.K2 * e3(d2_exact(pc, spos[cand_sorted[cs]], g.L, g.half)) < g.A6 * ii(i0);
            if (__builtin_amdgcn_readfirstlane((int)inside)) continue;
        }
        int64_t found = m;
        if constexpr (BINS) {
            // members per radial bin, then their inclusive prefix in place
            for (int k = tid; k < kRadBins; k += NT) s_rb[k] = 0u;
            __syncthreads();
            for_members<NT>(m, start, mem, spos, pc, g,
                            [&](double e) { atomicAdd(&s_rb[rbin_of(e, g.rbin)], 1u); });
            __syncthreads();
            constexpr int BI = kRadBins / NT;
            uint32_t v[BI];
            uint32_t sum = 0;
#pragma unroll
            for (int u = 0; u < BI; u++) {
                v[u] = s_rb[tid * BI + u];
                sum += v[u];
            }
            uint32_t tot;
            uint32_t P = block_excl<NT>(sum, s_red, &tot);
#pragma unroll
            for (int u = 0; u < BI; u++) {
                P += v[u];
                s_rb[tid * BI + u] = P;
            }
            __syncthreads();
            for (int j0 = 0; found == m;) {
                // the innermost occupied bin from j0 on that is not passed over
                int jb = 0x7fffffff;
                for (int j = j0 + tid; j < kRadBins; j += NT) {
                    const uint32_t Cj = j ? s_rb[j - 1] : 0u;
                    if (s_rb[j] > Cj && !(g.K2 * e3(rbin_edge2(j, g.rbin)) <= ii(Cj))) {
                        jb = j;
                        break;
                    }
                }
                const int js = block_min<NT>(jb, s_min);
                if (js == 0x7fffffff) break;  // no crossing inside the group
                const int64_t C = js ? s_rb[js - 1] : 0u;
                const int64_t cnt = (int64_t)s_rb[js] - C;
                const double lo = js ? rbin_edge2(js - 1, g.rbin) : -1.0, hi = rbin_edge2(js, g.rbin);
                uint32_t run = 0;
                for (int64_t w0 = 0; w0 < cnt && found == m; w0 += HL) {
                    const int64_t w1 = w0 + HL < cnt ? w0 + HL : cnt;
                    for (int64_t k = tid; k < w1 - w0; k += NT) s_hist[k] = 0u;
                    __syncthreads();
                    for_members<NT>(m, start, mem, spos, pc, g, [&](double e) {
                        if (e >= lo && e < hi) {
                            int64_t k = bucket_of(g.K2 * e3(e), m) - C;
                            k = k < 0 ? 0 : k;
                            if (k >= w0 && k < w1) atomicAdd(&s_hist[k - w0], 1u);
                        }
                    });
                    __syncthreads();
                    const int64_t t = first_crossing<NT>(s_hist, w0, w1, C, m, run, s_red, s_min);
                    if (t >= 0) found = C + t;
                }
                j0 = js + 1;
            }
        } else {
            // the buckets [w0, w1) each, and those beyond, 2^sh together
            uint32_t run = 0;  // C before w0
            for (int64_t w0 = 0; w0 < m && found == m;) {
                const int64_t w1 = m - w0 <= HL ? m : w0 + HL / 2;
                int sh = 0;
                while (m - w1 > (int64_t)(HL / 2) << sh) sh++;
                const int64_t nj = (m - w1 + (1ll << sh) - 1) >> sh;
                for (int64_t k = tid; k < w1 - w0 + nj; k += NT) s_hist[k] = 0u;
                __syncthreads();
                const double Tlo = w0 > 0 ? ii(w0 - 1) : -1.0, Thi = ii(m - 1);
                for_members<NT>(m, start, mem, spos, pc, g, [&](double e) {
                    const double T = g.K2 * e3(e);
                    if (!(T > Tlo && T <= Thi)) return;
                    const int64_t k = bucket_of(T, m);
                    atomicAdd(&s_hist[k < w1 ? k - w0 : w1 - w0 + ((k - w1) >> sh)], 1u);
                });
                __syncthreads();
                const int64_t t = first_crossing<NT>(s_hist, w0, w1, 0, m, run, s_red, s_min);
                if (t >= 0) found = t;
                const int64_t j = t >= 0 ? -1 : first_possible<NT>(s_hist + (w1 - w0), w1, nj, sh, run, s_red, s_min, &s_c);
                w0 = j < 0 ? m : w1 + (j << sh);
            }
        }
        if (tid == 0) {
            sti(enc + cr, (int32_t)found);
            if (ce - cs == 1u) {  // nothing to walk
                h_nuc[cs] = c;
                h_ienc[cs] = (int32_t)found;
                h_gid[cs] = gi;
                g_nh[gi] = 1;
            }
        }
        __syncthreads();  // the histogram and s_c are free for the next item
    }
}

// The walk over a group's candidates in descending density, a wavefront per
// group: 64 candidates at a time, one per lane, tested against the nuclei of the
// earlier ones; then the first lane left is accepted and the lanes after it are
// tested against it, until none is left.
__global__ __launch_bounds__(kBlock) void k_accept_walk(AcceptItems mid, AcceptItems big, Boxes bx,
                                                        const int32_t *__restrict__ gid_of,
                                                        const uint32_t *__restrict__ gcoff,
                                                        const int32_t *__restrict__ cand_sorted,
                                                        const float4 *__restrict__ spos,
                                                        const int32_t *__restrict__ enc, int32_t *h_nuc,
                                                        int32_t *h_ienc, int32_t *__restrict__ h_gid,
                                                        int32_t *__restrict__ g_nh) {
#pragma clang fp contract(off)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t nmid = *mid.firsts, count = nmid + *big.firsts;
    const uint32_t nw = gridDim.x * (kBlock / 64);
    for (uint32_t q = blockIdx.x * (kBlock / 64) + (uint32_t)wave; q < count; q += nw) {
        const uint32_t cs = (uint32_t)(q < nmid ? mid.list[q] : big.list[q - nmid]);
        const int c0 = cand_sorted[cs], gi = gid_of[c0];
        const uint32_t ce = gcoff[gi + 1];
        if (ce - cs == 1u) continue;  // settled with its candidate
        const Geo &g = bx.geo[__builtin_amdgcn_readfirstlane(box_of(bx, (uint32_t)c0))];
        uint32_t nh = 0;
        for (uint32_t b = cs; b < ce; b += 64) {
            const bool in = b + (uint32_t)lane < ce;
            const int c = in ? cand_sorted[b + (uint32_t)lane] : c0;
            const int32_t ic = in ? enc[b + (uint32_t)lane] : 0;
            const float4 pc = spos[c];
            bool el = in;
            for (uint32_t h = 0; h < nh; h++) {
                const double e = d2_exact(pc, spos[ldi(h_nuc + cs + h)], g.L, g.half);
                el = el && !(g.K2 * e3(e) < g.A6 * ii(ldi(h_ienc + cs + h)));
            }
            for (uint64_t left; (left = __ballot(el)) != 0ull; nh++) {
                const int L = (int)__builtin_ctzll(left);
                const int32_t in1 = lane_get(ic, L);
                const float4 pn = make_float4(lane_get(pc.x, L), lane_get(pc.y, L), lane_get(pc.z, L), 0.0f);
                if (lane == L) {
                    sti(h_nuc + cs + nh, c);
                    sti(h_ienc + cs + nh, ic);
                    h_gid[cs + nh] = gi;
                    el = false;
                }
                el = el && !(g.K2 * e3(d2_exact(pc, pn, g.L, g.half)) < g.A6 * ii(in1));
            }
            if (b + 64 < ce) __threadfence();  // the nuclei are read by the next 64
        }
        if (lane == 0) g_nh[gi] = (int32_t)nh;
    }
}

// --------------------------------------------------------------- assignment
// Step 3 as a per-particle fold over the group's halos in creation order, with
// the flat-rotation-curve enclosed density Delta_L1 R^2 / r^2 (Sec. 2.3.2)
// compared in cubed form: i_new^2 e_own^3 >= c^3 i_own^2 e_new^3.
__global__ __launch_bounds__(kBlock) void k_assign(int64_t n, Boxes bx, const int32_t *__restrict__ gid_of,
                                                   const uint32_t *__restrict__ gcoff,
                                                   const int32_t *__restrict__ g_nh,
                                                   const int32_t *__restrict__ h_nuc,
                                                   const int32_t *__restrict__ h_ienc,
                                                   const float4 *__restrict__ spos,
                                                   int32_t *__restrict__ owner,
                                                   uint32_t *__restrict__ h_count,
                                                   uint64_t *clock) {
#pragma clang fp contract(off)
    stamp(clock);
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int gi = i < n ? gid_of[i] : -1;
    int own = -1;
    if (gi >= 0) {
        const Geo &g = bx.geo[box_of(bx, (uint32_t)i)];
        const uint32_t cs = gcoff[gi];
        const int nh = g_nh[gi];
        const float4 pi = spos[i];
        double eown = 0.0, iown = 0.0;
        // the halos in creation order, four per round of loads (their
        // nuclei, then the nuclei's positions)
        for (int h0 = 0; h0 < nh; h0 += 4) {
            int nuc[4], ienc[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                nuc[u] = h0 + u < nh ? h_nuc[cs + h0 + u] : 0;
                ienc[u] = h0 + u < nh ? h_ienc[cs + h0 + u] : 0;
            }
            float4 pn[4];
#pragma unroll
            for (int u = 0; u < 4; u++) pn[u] = h0 + u < nh ? spos[nuc[u]] : pi;
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (h0 + u >= nh) break;
                const double e = d2_exact(pi, pn[u], g.L, g.half);
                const double ih = ii(ienc[u]);
                if (!(g.K2 * e3(e) < ih)) continue;
                bool take;
                if (own < 0) {
                    take = true;
                } else {
                    const double lhs = ih * e3(eown);
                    const double rhs = (g.C3 * iown) * e3(e);
                    take = lhs >= rhs;
                }
                if (take) {
                    own = (int)cs + h0 + u;
                    eown = e;
                    iown = ih;
                }
            }
        }
    }
    const WaveRun r = wave_run(own);
    if (own >= 0 && r.rank == 0) atomicAdd(&h_count[own], (uint32_t)r.len);
    if (i < n) owner[i] = own;
}

// ------------------------------------------------------------------- output

__global__ __launch_bounds__(kBlock) void k_out_flags(int64_t NC, Boxes bx, const int32_t *__restrict__ h_nuc,
                                                      const uint32_t *__restrict__ h_count,
                                                      const float4 *__restrict__ spos,
                                                      uint32_t *__restrict__ tflag,
                                                      int32_t *__restrict__ h_label,
                                                      int32_t *__restrict__ counters,
                                                      uint64_t *clock) {
    stamp(clock);
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int nuc = s < NC ? h_nuc[s] : -1;
    const uint64_t b = __ballot(nuc >= 0);
    if ((threadIdx.x & 63) == 0 && b) atomicAdd(&counters[2], __popcll(b));
    if (s >= NC) return;
    // the label every member of this halo gets: 1 + its nucleus's index in
    // the box when the halo is kept, else 0
    int32_t lab = 0;
    if (nuc >= 0) {
        const Geo &g = bx.geo[box_of(bx, (uint32_t)nuc)];
        if (h_count[s] >= (uint32_t)g.n_l1_min) {
            const uint32_t o = orig_of(spos[nuc]);
            atomicOr(&tflag[o >> 5], 1u << (o & 31u));
            lab = (int32_t)(o - g.orig_base) + 1;
        }
    }
    h_label[s] = lab;
}

// Kept halos with a nucleus below original index o: their bits before o's word
// (tpos, the prefix sum of the words' set bits) and below o in it.
__device__ __forceinline__ uint32_t table_pos(const uint32_t *__restrict__ tflag, const uint32_t *__restrict__ tpos,
                                              uint32_t o) {
    return tpos[o >> 5] + (uint32_t)__popc(tflag[o >> 5] & ((1u << (o & 31u)) - 1u));
}

// Rows of the halo table of every box: the kept halos are flagged at their
// nucleus's original index, so a box's rows are the flags in its index range.
// One workgroup, with the last words that the host reads.
__global__ __launch_bounds__(kBlock) void k_finish(Boxes bx, const uint32_t *__restrict__ tflag,
                                                   const uint32_t *__restrict__ tpos, WordSrc src, int k,
                                                   uint32_t *host, int64_t *rows, uint64_t *clock) {
    stamp(clock);
    for (int b = threadIdx.x; b < bx.nbox; b += blockDim.x)
        __hip_atomic_store(rows + b,
                           (int64_t)table_pos(tflag, tpos, bx.base[b + 1]) -
                               (int64_t)table_pos(tflag, tpos, bx.base[b]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const int t = threadIdx.x;
    if (t < k) __hip_atomic_store(host + t, *src.p[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A halo's row in its box's table (ascending id); a box whose rows exceed its
// table's capacity gets none written.  Ids and labels are box-local.
__global__ __launch_bounds__(kBlock) void k_out_table(int64_t NC, Boxes bx, const int32_t *__restrict__ h_nuc,
                                                      const int32_t *__restrict__ h_ienc,
                                                      const int32_t *__restrict__ h_gid,
                                                      const uint32_t *__restrict__ h_count,
                                                      const int32_t *__restrict__ g_label,
                                                      const float4 *__restrict__ spos,
                                                      const uint32_t *__restrict__ tflag,
                                                      const uint32_t *__restrict__ tpos) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= NC) return;
    int nuc = h_nuc[s];
    if (nuc < 0) return;
    const int box = box_of(bx, (uint32_t)nuc);
    const Geo &g = bx.geo[box];
    if (h_count[s] < (uint32_t)g.n_l1_min || !g.halos) return;
    const uint32_t b0 = table_pos(tflag, tpos, bx.base[box]);
    if ((int64_t)(table_pos(tflag, tpos, bx.base[box + 1]) - b0) > g.halo_cap) return;
    float4 p = spos[nuc];
    uint32_t o = orig_of(p);
    const int32_t lo = (int32_t)(o - g.orig_base);
    hf_halo h;
    h.id = lo + 1;
    h.nucleus = lo;
    h.l0_id = g_label[h_gid[s]] - (int32_t)g.orig_base;
    h.n = (int32_t)h_count[s];
    h.n_enclosed = h_ienc[s];
    h.x = p.x;
    h.y = p.y;
    h.z = p.z;
    h.r = (float)cbrt((double)h_ienc[s] / g.K);
    h.mass = (float)h_count[s] * g.particle_mass;
    g.halos[table_pos(tflag, tpos, o) - b0] = h;
}

// Only the halo labels to return: halo_id was filled with 0, and only the
// members of kept halos are written (scattered stores into the input order,
// so the fewer the better; their original index is read only for them).
__global__ __launch_bounds__(kBlock) void k_out_particles(int64_t n, const int32_t *__restrict__ owner,
                                                          const int32_t *__restrict__ h_label,
                                                          const float4 *__restrict__ spos,
                                                          int32_t *__restrict__ halo_id) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int own = owner[i];
    const int32_t lab = own >= 0 ? h_label[own] : 0;
    if (lab) halo_id[orig_of(spos[i])] = lab;
}

// With more than the halo labels to return: the record (density, L0 label,
// halo label) of every sorted particle stored at its original index, one
// scattered 16-byte store (one cache line) per particle instead of one per
// output array; k_out_split then writes the arrays in input order.
__global__ __launch_bounds__(kBlock) void k_out_records(int64_t n, Boxes bx, const int32_t *__restrict__ owner,
                                                        const int32_t *__restrict__ h_label,
                                                        const int32_t *__restrict__ gkey,
                                                        const float4 *__restrict__ spos,
                                                        const float *__restrict__ dens_s,
                                                        uint4 *__restrict__ rec) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int own = owner[i];
    const int32_t lab = own >= 0 ? h_label[own] : 0;
    const int32_t key = gkey[i];
    const Geo &g = bx.geo[box_of(bx, (uint32_t)i)];
    const int32_t l0 = key < 0 ? 0 : key + 1 - (int32_t)g.orig_base;
    rec[orig_of(spos[i])] = make_uint4(__float_as_uint(dens_s[i]), (uint32_t)l0, (uint32_t)lab, 0u);
}

__global__ __launch_bounds__(kBlock) void k_out_split(int64_t n, const uint4 *__restrict__ rec,
                                                      float *__restrict__ dens_out, int32_t *__restrict__ l0_out,
                                                      int32_t *__restrict__ halo_id) {
    int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= n) return;
    const uint4 r = rec[o];
    if (dens_out) dens_out[o] = __uint_as_float(r.x);
    if (l0_out) l0_out[o] = (int32_t)r.y;
    halo_id[o] = (int32_t)r.z;
}

// On large inputs the records take the way of a sort instead: partitioned by
// their original index into runs of kOutBucket, one or two passes, and then put
// in place in LDS.  A bucket's start is known (every index comes once), so a
// tile needs no counting pass: it takes its share of each bucket by an atomic.
// Scattered 16-byte records go to memory as 32-byte sectors all over it: 410 us
// and 98 for the split on the 256^3 box, 231 and 115 with the partition; 6.2 and
// 0.67 ms on the 512^3 box, 2.2 (two passes) and 0.71.  Below about 3 million
// particles the records stay in the memory-side cache and the scatter is faster
// (2^21: the output stage 58 us against 65; 2^22: 127 against 106).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // a record in registers
constexpr int kOutTile = 4096, kOutThreads = 512, kOutPer = kOutTile / kOutThreads;
constexpr int kOutBits = 14, kOutBucket = 1 << kOutBits;
constexpr int kOutBins = 1024;  // buckets of one pass at most
constexpr int64_t kOutPartLeast = (int64_t)1 << 22;

// One pass: records (density, L0 label, halo label, original index) of a tile
// into the buckets of 2^shift indices (first pass: from the sorted arrays; else
// from `in`, whose runs of 2^from indices hold whole tiles).
template <bool kFirst>
__global__ __launch_bounds__(kOutThreads, 4) void k_out_part(int64_t n, Boxes bx, const int32_t *__restrict__ owner,
                                                          const int32_t *__restrict__ h_label,
                                                          const int32_t *__restrict__ gkey,
                                                          const float4 *__restrict__ spos,
                                                          const float *__restrict__ dens_s,
                                                          const u32x4 *__restrict__ in, int from, int shift,
                                                          uint32_t *__restrict__ cursor, u32x4 *__restrict__ out) {
    __shared__ u32x4 s_rec[kOutTile];
    __shared__ uint32_t s_off[kOutBins], s_base[kOutBins];
    static_assert(kOutBins == 2 * kOutThreads, "two buckets per thread");
    const int64_t t0 = (int64_t)xcd_block() * kOutTile;
    // the tile's first possible bucket
    const uint32_t b0 = kFirst ? 0u : (uint32_t)(t0 >> from) << (from - shift);
    s_off[2 * threadIdx.x] = 0u;
    s_off[2 * threadIdx.x + 1] = 0u;
    __syncthreads();
    u32x4 rec[kOutPer];
    if (kFirst) {
        int32_t own[kOutPer], key[kOutPer];
#pragma unroll
        for (int k = 0; k < kOutPer; k++) {
            const int64_t i = t0 + k * kOutThreads + threadIdx.x, ic = i < n ? i : n - 1;
            own[k] = owner[ic];
            key[k] = gkey[ic];
            rec[k].x = __float_as_uint(dens_s[ic]);
            rec[k].w = orig_of(spos[ic]);
        }
#pragma unroll
        for (int k = 0; k < kOutPer; k++) {
            rec[k].y = key[k] < 0 ? 0u : (uint32_t)key[k] + 1u;
            rec[k].z = own[k] >= 0 ? (uint32_t)h_label[own[k]] : 0u;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kOutPer; k++) {
            const int64_t i = t0 + k * kOutThreads + threadIdx.x;
            rec[k] = in[i < n ? i : n - 1];
        }
    }
    uint32_t rank[kOutPer];
#pragma unroll
    for (int k = 0; k < kOutPer; k++)
        if (t0 + k * kOutThreads + threadIdx.x < n) rank[k] = atomicAdd(&s_off[(rec[k].w >> shift) - b0], 1u);
    __syncthreads();
    const uint32_t c0 = s_off[2 * threadIdx.x], c1 = s_off[2 * threadIdx.x + 1];
    uint32_t total;
    const uint32_t pre = block_excl_scan<kOutThreads>(c0 + c1, &total);
    const uint32_t b = b0 + 2u * threadIdx.x;
    s_off[2 * threadIdx.x] = pre;
    s_off[2 * threadIdx.x + 1] = pre + c0;
    if (c0) s_base[2 * threadIdx.x] = (b << shift) + atomicAdd(cursor + b, c0) - pre;
    if (c1) s_base[2 * threadIdx.x + 1] = ((b + 1u) << shift) + atomicAdd(cursor + b + 1u, c1) - (pre + c0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kOutPer; k++)
        if (t0 + k * kOutThreads + threadIdx.x < n) s_rec[s_off[(rec[k].w >> shift) - b0] + rank[k]] = rec[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kOutPer; k++) {
        const uint32_t j = k * kOutThreads + threadIdx.x;
        if (j < total) {
            u32x4 q = s_rec[j];
            // the L0 label in its box's numbering (a box holds the same indices
            // in input and in sorted order)
            if (kFirst && q.y) q.y -= (uint32_t)bx.geo[box_of(bx, q.w)].orig_base;
            out[s_base[(q.w >> shift) - b0] + j] = q;
        }
    }
}

// The records of a bucket to the output arrays, each put in order in LDS.
__global__ __launch_bounds__(1024) void k_out_place(int64_t n, const u32x4 *__restrict__ rec,
                                                    float *__restrict__ dens_out, int32_t *__restrict__ l0_out,
                                                    int32_t *__restrict__ halo_id) {
    __shared__ uint32_t s_val[kOutBucket];
    constexpr int kPer = kOutBucket / 1024;
    const int64_t o0 = (int64_t)xcd_block() * kOutBucket;
    const int m = (int)min((int64_t)kOutBucket, n - o0);
    u32x4 q[kPer];
#pragma unroll
    for (int k = 0; k < kPer; k++) {
        const int j = k * 1024 + threadIdx.x;
        q[k] = j < m ? rec[o0 + j] : u32x4{0u, 0u, 0u, 0u};
    }
    auto place = [&](auto pick, uint32_t *to) {
#pragma unroll
        for (int k = 0; k < kPer; k++)
            if (k * 1024 + (int)threadIdx.x < m) s_val[q[k].w & (uint32_t)(kOutBucket - 1)] = pick(q[k]);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int j = k * 1024 + threadIdx.x;
            if (j < m) to[o0 + j] = s_val[j];
        }
        __syncthreads();
    };
    if (dens_out) place([](const u32x4 &x) { return x.x; }, reinterpret_cast<uint32_t *>(dens_out));
    if (l0_out) place([](const u32x4 &x) { return x.y; }, reinterpret_cast<uint32_t *>(l0_out));
    place([](const u32x4 &x) { return x.z; }, reinterpret_cast<uint32_t *>(halo_id));
}

// ------------------------------------------------------------ group order
// Members collected into group order (Sec. 2.3.5): the particles sorted by the
// table row of their halo (particles of no halo after the last row), ascending
// original index within a row.  The paper sweeps the particles with in-place
// partitions, the largest halo and the unassigned ones first; here one stable
// sort by row gives every run at once.

// key = (row, original index); row = nrows for particles of no halo.  halo_id
// is in original order with labels 1 + nucleus index; tpos maps a kept
// nucleus to its table row.
__global__ __launch_bounds__(kBlock) void k_order_keys(int64_t n, int64_t nrows,
                                                       const int32_t *__restrict__ halo_id,
                                                       const uint32_t *__restrict__ tflag,
                                                       const uint32_t *__restrict__ tpos,
                                                       uint64_t *__restrict__ keys) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t h = halo_id[i];
    const uint64_t row = h > 0 ? (uint64_t)table_pos(tflag, tpos, (uint32_t)(h - 1)) : (uint64_t)nrows;
    keys[i] = (row << 32) | (uint64_t)i;
}

// members[t] from the sorted keys; halo_start[r] = first position of row r
// (the rows between two consecutive keys' rows start at the later key).
__global__ __launch_bounds__(kBlock) void k_order_out(int64_t n, int64_t nrows, const uint64_t *__restrict__ keys,
                                                      int32_t *__restrict__ members,
                                                      int64_t *__restrict__ halo_start) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t > n) return;
    if (t < n) members[t] = (int32_t)(keys[t] & 0xffffffffu);
    const int64_t rp = t > 0 ? (int64_t)(keys[t - 1] >> 32) : -1;
    const int64_t rc = t < n ? (int64_t)(keys[t] >> 32) : nrows + 1;
    for (int64_t r = rp + 1; r <= rc && r <= nrows; r++) halo_start[r] = t;
}

}  // namespace

void launch_segment_totals(int64_t n, Work &w, hipStream_t s) {
    const int64_t tiles = scan_tiles(n);
    uint32_t *msum = w.scan_tmp, *gsum = w.scan_tmp + tiles;
    hipLaunchKernelGGL(k_seg_sums, dim3((unsigned)tiles), dim3(kBlock), 0, s, n, w.gcnt, msum, gsum,
                       w.clock + kClockSegment);
    hipLaunchKernelGGL(k_seg_totals, dim3(1), dim3(kBlock), 0, s, tiles, msum, gsum, w.counters);
}

void launch_segment(int64_t n, Work &w, hipStream_t s) {
    const int64_t tiles = scan_tiles(n);
    uint32_t *msum = w.scan_tmp, *gsum = w.scan_tmp + tiles;
    hipLaunchKernelGGL(k_seg_sums, dim3((unsigned)tiles), dim3(kBlock), 0, s, n, w.gcnt, msum, gsum,
                       w.clock + kClockSegment);
    const bool scanned = scan_sums(w.scan_tmp, tiles, tiles, 2, s);
    // flags of the extent check in h_ienc (free until the acceptance fills it)
    hipLaunchKernelGGL(k_seg_offsets, dim3((unsigned)tiles), dim3(kBlock), 0, s, n, w.gcnt, msum, gsum, scanned,
                       w.goff, w.gidx, w.g_start, w.g_size, w.g_label, w.gccnt, w.gcfill, w.g_nh, w.h_ienc,
                       w.tflag, candidates_clear(n, w), w.counters);
    hipLaunchKernelGGL(k_seg_scatter, grid(n), dim3(kBlock), 0, s, n, w.gkey, w.goff, w.gidx, w.gcnt,
                       w.mem, w.gid_of);
}

void launch_extent(int64_t n, const Boxes &bx, Work &w, hipStream_t s) {
    // flags per group in h_ienc (zeroed with the group table) and the flagged
    // groups in glist (both free until the candidate stage), their count in
    // counters[12]; member and group counts are read on the device
    hipLaunchKernelGGL(k_extent_far, grid(n), dim3(kBlock), 0, s, w.counters + kCntMembers, bx, w.mem, w.gid_of,
                       w.g_start, w.spos, w.h_ienc, w.glist, reinterpret_cast<uint32_t *>(w.counters + 12));
    const int64_t blocks = n / 64 + 1;
    hipLaunchKernelGGL(k_extent_span, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(kBlock), 0, s,
                       reinterpret_cast<const uint32_t *>(w.counters + 12), bx, w.glist, w.g_start, w.g_size,
                       w.mem, w.spos, w.err);
}

static int bits_for(int64_t x) {
    int b = 1;
    while (b < 32 && (x >> b) != 0) b++;
    return b;
}

// A group's other candidates are evaluated beside its densest one, which costs
// nothing but idle compute units while they are few, and halves the time where
// they are nuclei of their own (groups of 40 000 in pairs: 121 us, 216 one after
// the other); but those inside its radius, nearly all in a large group with one
// centre, are evaluated for nothing.  By the histogram that is two passes over the
// group each: 250 000 members with 152 such candidates 534 us together and 604
// after it, 500 000 with 429 of them 1652 and 1187.  By the radial bins it is a
// pass for every bin out to a far crossing: 15 000 members in merging balls 103 us
// together and 163 after it, 30 000 with four such candidates 353 and 80, 500 000
// with 429 9.53 ms and 1.19.
constexpr int kLateHist = 4 * kHistBig, kLateBins = 16384;
int accept_late(const Work &w) { return w.radius_bins ? kLateBins : kLateHist; }

void launch_accept(int64_t n, int64_t G, int64_t NC, int64_t M, const Boxes &bx, Work &w, hipStream_t s) {
    // groups with candidates (at most min(G, NC)): those of one candidate and few
    // particles one wavefront each; the candidates of the others are listed (in
    // scratch arrays, which hold an entry per particle), evaluated by one workgroup
    // each and walked by one wavefront per group.  Persistent grids that stride over the lists: as many wavefronts
    // (six per SIMD) or workgroups (their LDS) as fit on the chip, and no more
    // than there are entries.  A group of kHistMid particles needs as many
    // members.  The counts are zero since the call began.
    const int64_t bound = G < NC ? G : NC;
    if (bound <= 0) return;
    auto counter = [&](int k) { return reinterpret_cast<uint32_t *>(w.counters + k); };
    const AcceptItems mid{reinterpret_cast<int32_t *>(w.tmp_a), counter(kCntMidFirst), counter(kCntMidRest), (uint32_t)n};
    const AcceptItems big{reinterpret_cast<int32_t *>(w.tmp_b), counter(kCntBigFirst), counter(kCntBigRest), (uint32_t)n};
    const AcceptItems late{reinterpret_cast<int32_t *>(w.tmp_d), counter(kCntLateListed), nullptr, (uint32_t)n};
    int32_t *enc = reinterpret_cast<int32_t *>(w.tmp_c);
    const int64_t ncu = w.ncu > 0 ? w.ncu : 1;
    auto cap = [](int64_t a, int64_t b) { return (unsigned)(a < b ? a : b); };
    const bool bins = w.radius_bins;
    // with few candidates every one gets 1024 threads, and a launch less (20 000
    // particles, 53 candidates: the second launch cost 5 us)
    const bool few = NC <= 4 * ncu;
    hipLaunchKernelGGL(k_accept_small, dim3(cap((bound + kBlock / 64 - 1) / (kBlock / 64), 6 * ncu)), dim3(kBlock),
                       0, s, counter(kCntListed), bins, few ? 0 : kHistMid, bx, w.glist, w.g_start, w.g_size, w.gcoff, w.cand_sorted,
                       w.mem, w.spos, w.h_nuc, w.h_ienc, w.h_gid, w.g_nh, mid, big, late, accept_late(w), enc,
                       w.clock + kClockAccept);
    if (!few)
        hipLaunchKernelGGL((bins ? k_accept_eval<kBlock, kHistMid, true> : k_accept_eval<kBlock, kHistMid, false>),
                           dim3(cap(NC, 4 * ncu)), dim3(kBlock), 0, s, mid, bx, w.gid_of, w.g_start, w.g_size, w.gcoff,
                           w.cand_sorted, w.mem, w.spos, enc, w.h_nuc, w.h_ienc, w.h_gid, w.g_nh);
    if (few || M >= kHistMid)
        hipLaunchKernelGGL((bins ? k_accept_eval<1024, kHistBig, true> : k_accept_eval<1024, kHistBig, false>),
                           dim3(cap(NC, ncu)), dim3(1024), 0, s, big, bx, w.gid_of, w.g_start, w.g_size, w.gcoff,
                           w.cand_sorted, w.mem, w.spos, enc, w.h_nuc, w.h_ienc, w.h_gid, w.g_nh);
    if (w.nlate > 0)
        hipLaunchKernelGGL((bins ? k_accept_eval<1024, kHistBig, true> : k_accept_eval<1024, kHistBig, false>),
                           dim3(cap(w.nlate, ncu)), dim3(1024), 0, s, late, bx, w.gid_of, w.g_start, w.g_size, w.gcoff,
                           w.cand_sorted, w.mem, w.spos, enc, w.h_nuc, w.h_ienc, w.h_gid, w.g_nh);
    // groups of two candidates at least
    if (NC > 1)
        hipLaunchKernelGGL(k_accept_walk, dim3(cap((bound + kBlock / 64 - 1) / (kBlock / 64), 6 * ncu)), dim3(kBlock), 0,
                           s, mid, big, bx, w.gid_of, w.gcoff, w.cand_sorted, w.spos, enc, w.h_nuc, w.h_ienc, w.h_gid,
                           w.g_nh);
}

void launch_assign(int64_t n, const Boxes &bx, Work &w, hipStream_t s) {
    hipLaunchKernelGGL(k_assign, grid(n), dim3(kBlock), 0, s, n, bx, w.gid_of, w.gcoff, w.g_nh, w.h_nuc,
                       w.h_ienc, w.spos, w.owner, w.h_count, w.clock + kClockAssign);
}

void launch_output_flags(int64_t n, int64_t NC, const Boxes &bx, Work &w, hipStream_t s) {
    // the table-row bits were zeroed with the group table
    if (NC > 0)
        // the candidates' member labels go to the hard-case list (free after
        // the candidate stage)
        hipLaunchKernelGGL(k_out_flags, grid(NC), dim3(kBlock), 0, s, NC, bx, w.h_nuc, w.h_count, w.spos,
                           w.tflag, w.hardlist, w.counters, w.clock + kClockOutput);
    scan_bits_u32(w.tflag, w.tpos, n / 32 + 1, w.scan_tmp, s);
}

void launch_output(int64_t n, int64_t NC, const Boxes &bx, Work &w, int32_t *halo_id, int32_t *l0_out,
                   float *dens_out, hipStream_t s) {
    if (NC > 0)
        hipLaunchKernelGGL(k_out_table, grid(NC), dim3(kBlock), 0, s, NC, bx, w.h_nuc, w.h_ienc, w.h_gid,
                           w.h_count, w.g_label, w.spos, w.tflag, w.tpos);
    if (!l0_out && !dens_out) {
        fill_i32(halo_id, 0, n, s);
        hipLaunchKernelGGL(k_out_particles, grid(n), dim3(kBlock), 0, s, n, w.owner, w.hardlist, w.spos,
                           halo_id);
        return;
    }
    // records in the radix key block (16 n bytes, free at this point)
    if (n >= kOutPartLeast) {
        u32x4 *rec = reinterpret_cast<u32x4 *>(w.rkey[0]);
        const dim3 tiles((unsigned)((n + kOutTile - 1) / kOutTile));
        const int64_t buckets = (n + kOutBucket - 1) / kOutBucket;
        // the cursors in the radix sort's payload, those of a first pass behind
        // the others'; its records in the scratch run of 4 (n + 1) words
        uint32_t *cursor = w.rval[0];
        if (buckets <= kOutBins) {
            fill_u32(cursor, 0u, buckets, s);
            hipLaunchKernelGGL(k_out_part<true>, tiles, dim3(kOutThreads), 0, s, n, bx, w.owner, w.hardlist, w.gkey,
                               w.spos, w.dens_s, nullptr, 0, kOutBits, cursor, rec);
        } else {
            // two passes of about equally many bits
            const int bits = bits_for(buckets - 1), from = kOutBits + bits / 2;
            const int64_t coarse = ((n - 1) >> from) + 1;
            u32x4 *half = reinterpret_cast<u32x4 *>(w.tmp_a);
            fill_u32(cursor, 0u, buckets + coarse, s);
            hipLaunchKernelGGL(k_out_part<true>, tiles, dim3(kOutThreads), 0, s, n, bx, w.owner, w.hardlist, w.gkey,
                               w.spos, w.dens_s, nullptr, 0, from, cursor + buckets, half);
            hipLaunchKernelGGL(k_out_part<false>, tiles, dim3(kOutThreads), 0, s, n, bx, nullptr, nullptr, nullptr,
                               nullptr, nullptr, half, from, kOutBits, cursor, rec);
        }
        hipLaunchKernelGGL(k_out_place, dim3((unsigned)buckets), dim3(1024), 0, s, n, rec, dens_out, l0_out, halo_id);
        return;
    }
    uint4 *rec = reinterpret_cast<uint4 *>(w.rkey[0]);
    hipLaunchKernelGGL(k_out_records, grid(n), dim3(kBlock), 0, s, n, bx, w.owner, w.hardlist, w.gkey, w.spos,
                       w.dens_s, rec);
    hipLaunchKernelGGL(k_out_split, grid(n), dim3(kBlock), 0, s, n, rec, dens_out, l0_out, halo_id);
}

void launch_finish(const Boxes &bx, const WordSrc &src, int k, Work &w, int64_t *rows, hipStream_t s) {
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kBlock), 0, s, bx, w.tflag, w.tpos, src, k, w.host, rows,
                       w.clock + kClockEnd);
}

void launch_group_order(int64_t n, int64_t nrows, const int32_t *halo_id, Work &w, int32_t *members,
                        int64_t *halo_start, hipStream_t s) {
    // the radix key arrays are free once the output is written
    hipLaunchKernelGGL(k_order_keys, grid(n), dim3(kBlock), 0, s, n, nrows, halo_id, w.tflag, w.tpos, w.rkey[0]);
    const uint64_t *sorted = radix_sort_keys(w.rkey[0], w.rkey[1], n, 32, bits_for(nrows + 1), w, s);
    hipLaunchKernelGGL(k_order_out, grid(n + 1), dim3(kBlock), 0, s, n, nrows, sorted, members, halo_start);
}

}  // namespace hf
