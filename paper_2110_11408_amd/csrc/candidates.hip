// Nucleus candidates (Sec. 2.2.2, steps 2 and 4): a member of an L0 group is a
// candidate when its density is at least the nucleation floor and no denser
// particle of the same group (eligible or not) lies within b.  "Denser" is the
// total order (density, then lower original index).  Candidacy depends only on
// the densities and the groups, so it is decided for all particles at once,
// before the sequential part of CompaSO.
//
// Two stages: most particles are settled by the densest particle of their own
// sub-cell, of their cell or of a face-adjacent sub-cell; the rest (sub-cell
// maxima and particles of sparse cells) are listed and searched by half a
// wavefront each, with pruning by the densest particle of every dense cell and
// sub-cell.
#include "hf_internal.h"
#include "scan_tile.h"

namespace hf {

namespace {

// Neighbour cell t of 27 in order of distance: own cell, the 6 face
// neighbours, the 12 edge neighbours, the 8 corners.
__constant__ int8_t kStencil[27] = {13, 4, 10, 12, 14, 16, 22, 1,  3,  5,  7,  9,  11, 15,
                                    17, 19, 21, 23, 25, 0, 2,  6,  8,  18, 20, 24, 26};

__device__ __forceinline__ void stencil_offset(int t, int &ox, int &oy, int &oz) {
    const int u = kStencil[t];
    ox = u % 3 - 1;
    oy = (u / 3) % 3 - 1;
    oz = u / 9 - 1;
}

// j is a denser particle of the same group within b.  Its group key and
// position are loaded together (one round trip: the searches wait on memory,
// not on arithmetic), and the distance is the canonical FP64 one.
__device__ __forceinline__ bool denser_within_b(int64_t j, const float *__restrict__ dens_s,
                                                const int32_t *__restrict__ gkey,
                                                const float4 *__restrict__ spos, int key, float di,
                                                uint32_t oi, const float4 &pi, const Geo &g) {
    const float dj = dens_s[j];
    const int kj = gkey[j];
    const float4 pj = spos[j];
    if (dj < di || kj != key) return false;
    if (!denser(dj, orig_of(pj), di, oi)) return false;
    return d2_exact(pi, pj, g.L, g.half) < g.b2;
}

// Densest particle of every sub-cell of a dense cell, as a packed key
// (density bits, inverted original index): larger key = denser in the total
// order (densities are >= 0, so their bit patterns order like the values).
__device__ __forceinline__ uint64_t dkey(float d, uint32_t orig) {
    return ((uint64_t)__float_as_uint(d) << 32) | (uint64_t)(0xffffffffu - orig);
}

// One wavefront per dense cell: the cell's particles are sorted by sub-cell,
// so each 64-particle step reduces the runs of equal sub-cells (maximum key
// and its particle) and the first lane of each run merges the result into the
// cell's row in LDS.  Entry nsub_max of the row (sub-cells end before it) is
// the densest particle of the whole cell.
constexpr int kSubMost = 216;  // 6^3 sub-cells at most
__global__ __launch_bounds__(kBlock) void k_submax_wave(int64_t ndc, Boxes bx,
                                                        const uint32_t *__restrict__ subtab,
                                                        const uint16_t *__restrict__ ssub,
                                                        const float *__restrict__ dens_s,
                                                        const float4 *__restrict__ spos,
                                                        uint64_t *__restrict__ submax,
                                                        int32_t *__restrict__ subarg,
                                                        uint64_t *clock) {
    stamp(clock);
    __shared__ uint64_t s_best[kBlock / 64][kSubMost];
    __shared__ int32_t s_arg[kBlock / 64][kSubMost];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t d = (int64_t)blockIdx.x * (kBlock / 64) + wave;
    if (d >= ndc) return;
    const int lane = threadIdx.x & 63;
    const int64_t row = d * (bx.nsub_max + 1);
    const uint32_t a = (uint32_t)__builtin_amdgcn_readfirstlane(subtab[row]);
    const int nsub = __builtin_amdgcn_readfirstlane(bx.geo[box_of(bx, a)].nsub);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane(subtab[row + nsub]);
    for (int v = lane; v < nsub; v += 64) {
        s_best[wave][v] = 0ull;
        s_arg[wave][v] = -1;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t j0 = a; j0 < b; j0 += 64) {
        const uint32_t j = j0 + (uint32_t)lane;
        const bool act = j < b;
        const int v = act ? (int)ssub[j] : -1 - lane;  // inactive lanes: runs of their own
        uint64_t kk = act ? dkey(dens_s[j], orig_of(spos[j])) : 0ull;
        int32_t jj = (int32_t)j;
        const WaveRun run = wave_run(v);
        const int end = run.head + run.len;
        for (int dd = 1; dd < 64; dd <<= 1) {
            const uint32_t olo = __shfl_down((uint32_t)kk, dd, 64), ohi = __shfl_down((uint32_t)(kk >> 32), dd, 64);
            const int32_t oj = __shfl_down(jj, dd, 64);
            const uint64_t ok = ((uint64_t)ohi << 32) | olo;
            if (lane + dd < end && ok > kk) {
                kk = ok;
                jj = oj;
            }
        }
        if (act && run.rank == 0 && (s_arg[wave][v] < 0 || kk > s_best[wave][v])) {
            s_best[wave][v] = kk;
            s_arg[wave][v] = jj;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
    }
    uint64_t top = 0ull;
    int32_t targ = -1;
    for (int v = lane; v < nsub; v += 64) {
        const uint64_t best = s_best[wave][v];
        const int32_t arg = s_arg[wave][v];
        submax[row + v] = best;
        subarg[row + v] = arg;
        if (arg >= 0 && (targ < 0 || best > top)) {
            top = best;
            targ = arg;
        }
    }
    for (int dd = 32; dd >= 1; dd >>= 1) {
        const uint32_t olo = __shfl_xor((uint32_t)top, dd, 64), ohi = __shfl_xor((uint32_t)(top >> 32), dd, 64);
        const int32_t oarg = __shfl_xor(targ, dd, 64);
        const uint64_t ok = ((uint64_t)ohi << 32) | olo;
        if (oarg >= 0 && (targ < 0 || ok > top)) {
            top = ok;
            targ = oarg;
        }
    }
    if (lane == 0) {
        submax[row + bx.nsub_max] = top;
        subarg[row + bx.nsub_max] = targ;
    }
}

// Stage 1, one thread per particle: a member at or above the floor that is not
// the densest particle of its sub-cell is decided at once when that densest
// particle belongs to its group and lies within b (the usual case inside an L0
// group, the sub-cell diagonal being below l).  A member that is its
// sub-cell's densest is decided in the same way by the densest particle of its
// cell, or when the densest particle of a face-adjacent sub-cell of the same
// cell is denser and in its group, where such sub-cells lie within b of each
// other entirely (s sqrt(6) < b).  Every other member at or above the floor is
// listed as a hard case.  The kernel waits on rounds of dependent loads: with the
// marks loaded next to the key, and the cell's densest particle tested in the
// round that a sub-cell's densest had free, it takes 190 us on the 256^3 box
// (248 before) and leaves 371 000 hard cases of 524 000 (k_cand_search 324 ->
// 236 us).
template <int kQuickPer>  // particles per thread
__global__ __launch_bounds__(kBlock) void k_cand_quick(int64_t n, Boxes bx,
                                                       const float4 *__restrict__ spos,
                                                       Marks marks, const uint16_t *__restrict__ ssub,
                                                       const uint64_t *__restrict__ submax,
                                                       const int32_t *__restrict__ subarg,
                                                       const float *__restrict__ dens_s,
                                                       const int32_t *__restrict__ gkey,
                                                       SegList hl,
                                                       uint64_t *clock) {
    stamp(clock);
    const int64_t i0 = (int64_t)xcd_block() * (kQuickPer * kBlock) + threadIdx.x;
    bool hard[kQuickPer], dense[kQuickPer];
    int key[kQuickPer], si[kQuickPer];
    int32_t idx[kQuickPer], own[kQuickPer], most[kQuickPer];
    uint32_t cell[kQuickPer];
    float di[kQuickPer];
    float4 pi[kQuickPer];
    // (the marks with the key and the density, so that a member saves a round of
    // loads)
#pragma unroll
    for (int u = 0; u < kQuickPer; u++) {
        const int64_t i = i0 + u * kBlock, ic = i < n ? i : n - 1;
        idx[u] = (int32_t)i;
        key[u] = i < n ? gkey[ic] : -1;
        di[u] = dens_s[ic];
        dense[u] = !is_sparse(marks, ic);
        si[u] = ssub[ic];
        cell[u] = dense_ordinal(marks, (uint32_t)ic);
    }
#pragma unroll
    for (int u = 0; u < kQuickPer; u++) {
        const int64_t i = i0 + u * kBlock, ic = i < n ? i : n - 1;
        hard[u] = key[u] >= 0 && (double)di[u] >= bx.geo[box_of(bx, (uint32_t)ic)].floor_nuc;
        dense[u] = dense[u] && hard[u];
        own[u] = most[u] = idx[u];
        if (dense[u]) {
            const int64_t base = (int64_t)cell[u] * (bx.nsub_max + 1);
            own[u] = subarg[base + si[u]];
            most[u] = subarg[base + bx.nsub_max];
            pi[u] = spos[i];
        }
    }
    // the maximum of i's sub-cell or, when that is i, of its cell, is denser than
    // i (the bit order of the key matches the values for the non-negative
    // densities the stage works on; checked anyway); its key, density and
    // position are loaded together
    int kt1[kQuickPer];
    float dt1[kQuickPer];
    float4 pt1[kQuickPer];
#pragma unroll
    for (int u = 0; u < kQuickPer; u++) {
        const int32_t top = own[u] != idx[u] ? own[u] : most[u];
        kt1[u] = -1;
        if (top != idx[u]) {
            kt1[u] = gkey[top];
            dt1[u] = dens_s[top];
            pt1[u] = spos[top];
        }
    }
#pragma unroll
    for (int u = 0; u < kQuickPer; u++) {
        if (!dense[u]) continue;
        const Geo &g = bx.geo[box_of(bx, (uint32_t)idx[u])];
        const uint32_t oi = orig_of(pi[u]);
        if (kt1[u] == key[u] && denser(dt1[u], orig_of(pt1[u]), di[u], oi) &&
            d2_exact(pi[u], pt1[u], g.L, g.half) < g.b2)
            hard[u] = false;
        // (the densest particle of the cell has no denser sub-cell next to it)
        if (hard[u] && own[u] == idx[u] && most[u] != idx[u] && g.face_sub_in_b) {
            const int64_t base = (int64_t)cell[u] * (bx.nsub_max + 1);
                // the six face-adjacent sub-cells at once: their maxima, then
                // the particles that hold them, then those particles' keys
                const int k = g.ksub;
                const int sz = div_small(si[u], 1.0f / (float)(k * k)), syx = si[u] - sz * k * k,
                          sy = div_small(syx, 1.0f / (float)k), sx = syx - sy * k;
                const uint64_t mykey = dkey(di[u], oi);
                int s2[6];
                uint64_t mx[6];
#pragma unroll
                for (int f = 0; f < 6; f++) {
                    const int ax = f >> 1, dir = (f & 1) ? 1 : -1;
                    const int nx = sx + (ax == 0 ? dir : 0), ny = sy + (ax == 1 ? dir : 0),
                              nz = sz + (ax == 2 ? dir : 0);
                    const bool in = nx >= 0 && nx < k && ny >= 0 && ny < k && nz >= 0 && nz < k;
                    s2[f] = in ? (nz * k + ny) * k + nx : -1;
                    mx[f] = in ? submax[base + s2[f]] : 0ull;
                }
                int32_t t2[6];
#pragma unroll
                for (int f = 0; f < 6; f++) t2[f] = mx[f] > mykey ? subarg[base + s2[f]] : -1;
                int kt[6];
                float dt[6];
                uint32_t ot[6];
#pragma unroll
                for (int f = 0; f < 6; f++) {
                    kt[f] = -1;
                    dt[f] = 0.0f;
                    ot[f] = 0u;
                    if (t2[f] >= 0) {
                        kt[f] = gkey[t2[f]];
                        dt[f] = dens_s[t2[f]];
                        ot[f] = orig_of(spos[t2[f]]);
                    }
                }
#pragma unroll
                for (int f = 0; f < 6; f++)
                    if (t2[f] >= 0 && kt[f] == key[u] && denser(dt[f], ot[f], di[u], oi)) hard[u] = false;
        }
    }
    seg_append<kQuickPer>(hl, hard, idx);
}

// Stage 2, half a wavefront per hard case: whether a denser particle of the
// group lies within b.  Each step is one round of loads over the 27 stencil
// cells (one per lane) or 32 sub-cells, and the search stops at the first
// denser particle:
//   the ranges of the stencil cells; the particles of the sparse ones (their
//   densities together, the denser ones in full);
//   the densest particle of every dense cell (a cell without a denser particle
//   is dropped: mostly all but a few);
//   the sub-cells of the cells left, 32 at a time: those within b that hold a
//   denser particle test their densest one, then the rest, a long sub-cell
//   with all lanes.
// The search is a chain of dependent loads, so what counts is the number of
// rounds a case takes and the cases in flight.  One thread per case for the
// own cell and then for the face neighbours (nine or more rounds per dense
// cell, the chain of a wavefront its longest case's) took 146 us on a box of
// 20 000 particles, 178 us on the 64^3 box and 455 us on the 256^3 one.
__global__ __launch_bounds__(kBlock) void k_cand_search(SegList hl, Boxes bx, const float4 *__restrict__ sloc,
                                                        const float4 *__restrict__ spos,
                                                        Cells cells, const uint32_t *__restrict__ subtab,
                                                        const uint64_t *__restrict__ submax,
                                                        const int32_t *__restrict__ subarg,
                                                        const float *__restrict__ dens_s,
                                                        const int32_t *__restrict__ gkey,
                                                        const int32_t *__restrict__ gid_of,
                                                        uint32_t *__restrict__ gccnt,
                                                        int32_t *__restrict__ nhard) {
    constexpr int kHalves = kBlock / 32;
    __shared__ int64_t s_base[kHalves][27];  // sub-table bases of a case's open dense cells
    __shared__ int8_t s_tt[kHalves][27];     // and their stencil order index
    const int hw = threadIdx.x >> 5, ln = threadIdx.x & 31, hsh = threadIdx.x & 32;
    auto hballot = [&](bool p) { return (uint32_t)(__ballot(p) >> hsh); };
    if (blockIdx.x == 0 && threadIdx.x < kSegs) {
        int32_t t = threadIdx.x < hl.nseg ? (int32_t)hl.count[threadIdx.x * kSegStride] : 0;
        for (int d = 32; d >= 1; d >>= 1) t += __shfl_xor(t, d, 64);
        if (threadIdx.x == 0) *nhard = t;
    }
    const SegShare sh = seg_share<32>(hl);
    const int tstride = bx.nsub_max + 1;
    for (uint32_t k = sh.k; k < sh.n; k += sh.step) {
        int32_t *const entry = hl.list + (int64_t)sh.seg * hl.cap + k;
        const int i = *entry;
        per_box(bx, box_of(bx, (uint32_t)i), [&](const Geo &g) {
        const int key = gkey[i];
        const float di = dens_s[i];
        const float4 li = sloc[i];
        const float4 pi = spos[i];
        const uint32_t oi = orig_of(pi);
        const uint64_t mykey = dkey(di, oi);
        int cx, cy, cz;
        cell_xyz(g, __float_as_uint(li.w), cx, cy, cz);
        bool found = false, dense = false;
        uint32_t number = 0;
        if (ln < 27) {
            int ox, oy, oz;
            stencil_offset(ln, ox, oy, oz);
            const float gx = ox < 0 ? li.x : (ox > 0 ? g.cellb - li.x : 0.0f);
            const float gy = oy < 0 ? li.y : (oy > 0 ? g.cellb - li.y : 0.0f);
            const float gz = oz < 0 ? li.z : (oz > 0 ? g.cellb - li.z : 0.0f);
            if (gx * gx + gy * gy + gz * gz < g.b2b_hi) {
                uint32_t a, b;
                number = cell_range(cells, cell_id(g, cx + ox, cy + oy, cz + oz), a, b);
                dense = b - a >= (uint32_t)kDenseMin;
                if (!dense) {
                    float dj[kDenseMin - 1];
#pragma unroll
                    for (int v = 0; v < kDenseMin - 1; v++) dj[v] = a + v < b ? dens_s[a + v] : -1.0f;
#pragma unroll
                    for (int v = 0; v < kDenseMin - 1; v++)
                        if (a + v < b && dj[v] >= di && (int)(a + v) != i && !found)
                            found = denser_within_b(a + v, dens_s, gkey, spos, key, di, oi, pi, g);
                }
            }
        }
        if (hballot(found)) return;
        bool open = false;
        int64_t base = 0;
        if (dense) {
            base = (int64_t)cells.dmap[number] * tstride;
            const uint64_t mx = submax[base + bx.nsub_max];
            const int32_t top = subarg[base + bx.nsub_max];
            open = mx > mykey;
            if (open) found = denser_within_b(top, dens_s, gkey, spos, key, di, oi, pi, g);
        }
        if (hballot(found)) return;
        const uint32_t om = hballot(open);
        if (open) {
            const int slot = __popc(om & ((1u << ln) - 1u));
            s_base[hw][slot] = base;
            s_tt[hw][slot] = (int8_t)ln;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        const int ks = g.ksub, nsub = g.nsub;
        const float subb = g.cellb / (float)ks;
        const float inv_nsub = 1.0f / (float)nsub, inv_k = 1.0f / (float)ks, inv_k2 = 1.0f / (float)(ks * ks);
        const int ntask = __popc(om) * nsub;
        for (int t0 = 0; t0 < ntask; t0 += 32) {
            const int tq = t0 + ln;
            uint32_t u0 = 0, u1 = 0;  // the sub-cell's particles still to be looked at
            int32_t top = -1;
            if (tq < ntask) {
                const int r = div_small(tq, inv_nsub), sl = tq - r * nsub;
                const int64_t row = s_base[hw][r] + sl;
                const uint64_t mx = submax[row];
                const int32_t arg = subarg[row];
                const uint32_t b0 = subtab[row], b1 = subtab[row + 1];
                if (mx > mykey) {
                    int ox, oy, oz;
                    stencil_offset(s_tt[hw][r], ox, oy, oz);
                    const float xs = li.x - (float)ox * g.cellb, ys = li.y - (float)oy * g.cellb,
                                zs = li.z - (float)oz * g.cellb;
                    const int sz = div_small(sl, inv_k2), syx = sl - sz * ks * ks, sy = div_small(syx, inv_k),
                              sx = syx - sy * ks;
                    const float ex = fmaxf(fmaxf(sx * subb - 1e-5f - xs, xs - (sx + 1) * subb - 1e-5f), 0.0f);
                    const float ey = fmaxf(fmaxf(sy * subb - 1e-5f - ys, ys - (sy + 1) * subb - 1e-5f), 0.0f);
                    const float ez = fmaxf(fmaxf(sz * subb - 1e-5f - zs, zs - (sz + 1) * subb - 1e-5f), 0.0f);
                    if (ex * ex + ey * ey + ez * ez < g.b2b_hi) {
                        top = arg;
                        found = denser_within_b(top, dens_s, gkey, spos, key, di, oi, pi, g);
                        u0 = b0;
                        u1 = b1;
                    }
                }
            }
            if (hballot(found)) break;
            // the rest of the sub-cells: short ones by their own lane, the
            // others by all lanes
            constexpr uint32_t kShort = 8;
            if (u1 - u0 <= kShort) {
                float dj[kShort];
#pragma unroll
                for (uint32_t v = 0; v < kShort; v++) dj[v] = u0 + v < u1 ? dens_s[u0 + v] : -1.0f;
#pragma unroll
                for (uint32_t v = 0; v < kShort; v++) {
                    const uint32_t j = u0 + v;
                    if (j < u1 && dj[v] >= di && (int32_t)j != top && (int)j != i && !found)
                        found = denser_within_b(j, dens_s, gkey, spos, key, di, oi, pi, g);
                }
            }
            for (uint32_t m = hballot(u1 - u0 > kShort); m && !hballot(found); m &= m - 1) {
                const int src = __ffs(m) - 1;
                const uint32_t c0 = __shfl(u0, src, 32), c1 = __shfl(u1, src, 32);
                for (uint32_t j0 = c0; j0 < c1 && !hballot(found); j0 += 32) {
                    const uint32_t j = j0 + (uint32_t)ln;
                    if (j < c1 && (int)j != i && dens_s[j] >= di)
                        found = denser_within_b(j, dens_s, gkey, spos, key, di, oi, pi, g);
                }
            }
            if (hballot(found)) break;
        }
        if (!hballot(found) && ln == 0) {
            // a candidate: marked in the list, counted for its group
            *entry = ~i;
            atomicAdd(&gccnt[gid_of[i]], 1u);
        }
        });
    }
}

// ------------------------------------------------------------ candidate lists
// Size classes of the groups with candidates: four per octave.
constexpr int kClasses = 128;
__device__ __forceinline__ int size_class(uint32_t m) {
    return (int)(__float_as_uint((float)m) >> 21) - (int)(0x3f800000u >> 21);
}

__global__ __launch_bounds__(kBlock) void k_gc_sums(const int32_t *__restrict__ groups_p,
                                                    const uint32_t *__restrict__ gccnt,
                                                    uint32_t *__restrict__ sums) {
    const int64_t G = *groups_p, base = (int64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
    if (base < G) tile_each(gccnt, base, G, [&](uint32_t x) { s += x; });
    const uint32_t tot = block_sum(s);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// First candidate of every group (gcoff[G] and counters[kCntCand]: their
// total), the number of groups with candidates per size class, and how many
// candidates of groups above `late` members are not their group's first.  The
// group count is read on the device.
__global__ __launch_bounds__(kBlock) void k_gc_offsets(const uint32_t *__restrict__ gccnt,
                                                       const int32_t *__restrict__ g_size,
                                                       const uint32_t *__restrict__ sums, bool scanned, int late,
                                                       uint32_t *__restrict__ gcoff,
                                                       uint32_t *__restrict__ nclass,
                                                       int32_t *__restrict__ counters) {
    __shared__ uint32_t buf[kScanLds];
    __shared__ uint32_t s_class[kClasses], s_late;
    const int64_t G = counters[kCntGroups], base = (int64_t)blockIdx.x * kScanTile;
    if (base >= G && blockIdx.x > 0) return;
    if (threadIdx.x < kClasses) s_class[threadIdx.x] = 0u;
    if (threadIdx.x == 0) s_late = 0u;
    uint32_t v[kScanItems];
    tile_load(gccnt, base, G, buf, v, [](uint32_t x) { return x; });
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) s += v[k];
    uint32_t tot;
    uint32_t run = block_excl_scan(s, &tot);
    const uint32_t toff = blockIdx.x > 0 ? tile_offset(sums, blockIdx.x, scanned) : 0u;
    run += toff;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        const int64_t g = base + (int64_t)threadIdx.x * kScanItems + k;
        if (g >= G) break;
        gcoff[g] = run;
        run += v[k];
        if (v[k] == 0u) continue;
        const int32_t m = g_size[g];
        atomicAdd(&s_class[size_class((uint32_t)m)], 1u);
        if (m > late && v[k] > 1u) atomicAdd(&s_late, v[k] - 1u);
    }
    __syncthreads();
    if (threadIdx.x < kClasses && s_class[threadIdx.x]) atomicAdd(&nclass[threadIdx.x], s_class[threadIdx.x]);
    if (threadIdx.x == 0 && s_late) atomicAdd(&counters[kCntLate], (int32_t)s_late);
    if (base + kScanTile >= G && threadIdx.x == 0) {
        gcoff[G] = toff + tot;
        counters[kCntCand] = (int32_t)(toff + tot);
    }
}

// The candidates of the hard-case list into their groups' slots (any order
// inside a group), with the slots' halo records cleared.
__global__ __launch_bounds__(kBlock) void k_cand_scatter(SegList hl, const int32_t *__restrict__ gid_of,
                                                         const uint32_t *__restrict__ gcoff,
                                                         uint32_t *__restrict__ gcfill,
                                                         int32_t *__restrict__ cand,
                                                         int32_t *__restrict__ h_nuc,
                                                         uint32_t *__restrict__ h_count) {
    const uint32_t seg = blockIdx.x % hl.nseg, nb = gridDim.x / hl.nseg;
    const uint32_t cnt = hl.count[seg * kSegStride];
    for (uint32_t k = (blockIdx.x / hl.nseg) * kBlock + threadIdx.x; k < cnt; k += nb * kBlock) {
        const int32_t e = hl.list[(int64_t)seg * hl.cap + k];
        if (e >= 0) continue;
        const int i = ~e, gi = gid_of[i];
        const uint32_t slot = gcoff[gi] + atomicAdd(&gcfill[gi], 1u);
        cand[slot] = i;
        h_nuc[slot] = -1;
        h_count[slot] = 0u;
    }
}

// Order candidates of a group by "denser" (density desc, original index asc):
// the rank of a candidate is the number of denser candidates in its group.
__global__ __launch_bounds__(kBlock) void k_cand_rank(const int32_t *__restrict__ ncand_p,
                                                      const int32_t *__restrict__ gid_of,
                                                      const uint32_t *__restrict__ gcoff,
                                                      const int32_t *__restrict__ cand,
                                                      const float *__restrict__ dens_s,
                                                      const float4 *__restrict__ spos,
                                                      int32_t *__restrict__ cand_sorted) {
    const int64_t NC = *ncand_p;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < NC;
         s += (int64_t)gridDim.x * blockDim.x) {
        const int me = cand[s];
        const int gi = gid_of[me];
        const uint32_t a = gcoff[gi], b = gcoff[gi + 1];
        const float dm = dens_s[me];
        const uint32_t om = orig_of(spos[me]);
        uint32_t rank = 0;
        for (uint32_t t = a; t < b; t++) {
            const int o = cand[t];
            rank += denser(dens_s[o], orig_of(spos[o]), dm, om) ? 1u : 0u;
        }
        cand_sorted[a + rank] = me;
    }
}

// The groups with candidates (of every box), the larger size classes first, so
// that the acceptance kernels start the longest walks first.  The order inside
// a class is that of arrival: nothing but the schedule depends on it, and the
// classes differ by a quarter octave (a radix sort by size, three to four
// passes of four launches, cost 60 us on a list of a few hundred groups).
__global__ __launch_bounds__(kBlock) void k_group_list(const uint32_t *__restrict__ gccnt,
                                                       const int32_t *__restrict__ g_size,
                                                       const uint32_t *__restrict__ nclass,
                                                       uint32_t *__restrict__ fill,
                                                       int32_t *__restrict__ glist,
                                                       int32_t *__restrict__ counters) {
    __shared__ uint32_t s_start[kClasses], s_cnt[kClasses], s_at[kClasses];
    const int64_t G = counters[kCntGroups];
    // larger classes first: class c starts after the classes above it
    const int rc = kClasses - 1 - (int)threadIdx.x;
    uint32_t tot;
    const uint32_t before = block_excl_scan(rc >= 0 ? nclass[rc] : 0u, &tot);
    if (rc >= 0) s_start[rc] = before;
    if (blockIdx.x == 0 && threadIdx.x == 0) counters[kCntListed] = (int32_t)tot;
    for (int64_t g0 = (int64_t)blockIdx.x * kBlock; g0 < G; g0 += (int64_t)gridDim.x * kBlock) {
        if (threadIdx.x < kClasses) s_cnt[threadIdx.x] = 0u;
        __syncthreads();
        const int64_t g = g0 + threadIdx.x;
        const bool in = g < G && gccnt[g] != 0u;
        int c = 0;
        uint32_t rank = 0;
        if (in) {
            c = size_class((uint32_t)g_size[g]);
            rank = atomicAdd(&s_cnt[c], 1u);
        }
        __syncthreads();
        if (threadIdx.x < kClasses && s_cnt[threadIdx.x])
            s_at[threadIdx.x] = atomicAdd(&fill[threadIdx.x], s_cnt[threadIdx.x]);
        __syncthreads();
        if (in) glist[s_start[c] + s_at[c] + rank] = (int32_t)g;
        __syncthreads();
    }
}

}  // namespace

SegClear candidates_clear(int64_t n, const Work &w) {
    // the counts of the hard-case segments, and the class counts and fills of
    // the group list in the scanned radix counts (257 words at least)
    static_assert(2 * kClasses <= 257, "class counts fit the smallest radix count array");
    return SegClear{{w.rhist, w.rscan}, {(int)(seg_list(n, w).nseg * kSegStride), 2 * kClasses}};
}

void launch_candidates(int64_t n, const Boxes &bx, Work &w, hipStream_t s) {
    if (w.ndcells > 0)
        hipLaunchKernelGGL(k_submax_wave, dim3((unsigned)((w.ndcells + kBlock / 64 - 1) / (kBlock / 64))),
                           dim3(kBlock), 0, s, w.ndcells, bx, w.subtab, w.ssub, w.dens_s, w.spos, w.submax,
                           w.subarg, w.clock + kClockCand);
    const SegList hl = seg_list(n, w);
    const int64_t per = list_per(n) * kBlock;
    hipLaunchKernelGGL(list_per(n) == 2 ? k_cand_quick<2> : k_cand_quick<1>, dim3((unsigned)((n + per - 1) / per)),
                       dim3(kBlock), 0, s, n, bx,
                       w.spos, w.marks, w.ssub, w.submax, w.subarg, w.dens_s, w.gkey, hl,
                       w.ndcells > 0 ? nullptr : w.clock + kClockCand);
    // half-wavefronts striding over the segments: as many as fit the chip (six
    // wavefronts per SIMD at 79 VGPRs), and no more than one per four particles
    // (one particle in thirty is a hard case); their total goes to a counter
    const unsigned blocks = seg_blocks(hl, n, 32, 4, 6 * (int64_t)(w.ncu > 0 ? w.ncu : 1));
    hipLaunchKernelGGL(k_cand_search, dim3(blocks), dim3(kBlock), 0, s, hl, bx, w.sloc, w.spos, w.cells,
                       w.subtab, w.submax, w.subarg, w.dens_s, w.gkey, w.gid_of, w.gccnt,
                       w.counters + kCntHard);
    const int64_t tiles = scan_tiles(n);  // of the groups: at most one per particle
    hipLaunchKernelGGL(k_gc_sums, dim3((unsigned)tiles), dim3(kBlock), 0, s, w.counters + kCntGroups, w.gccnt,
                       w.scan_tmp);
    const bool scanned = scan_sums(w.scan_tmp, tiles, tiles, 1, s);
    hipLaunchKernelGGL(k_gc_offsets, dim3((unsigned)tiles), dim3(kBlock), 0, s, w.gccnt, w.g_size, w.scan_tmp,
                       scanned, accept_late(w), w.gcoff, w.rscan, w.counters);
}

void launch_candidate_lists(int64_t n, Work &w, hipStream_t s) {
    // grids that stride over counts known on the device
    const SegList hl = seg_list(n, w);
    auto cap = [](int64_t want, int64_t most) { return (unsigned)(want < most ? want : most); };
    const unsigned per = cap((int64_t)hl.cap / (16 * kBlock) + 1, 16);
    hipLaunchKernelGGL(k_cand_scatter, dim3(hl.nseg * per), dim3(kBlock), 0, s, hl, w.gid_of, w.gcoff, w.gcfill,
                       w.cand, w.h_nuc, w.h_count);
    hipLaunchKernelGGL(k_cand_rank, dim3(cap(n / (64 * kBlock) + 1, 1024)), dim3(kBlock), 0, s,
                       w.counters + kCntCand, w.gid_of, w.gcoff, w.cand, w.dens_s, w.spos, w.cand_sorted);
    hipLaunchKernelGGL(k_group_list, dim3(cap(n / (32 * kBlock) + 1, 1024)), dim3(kBlock), 0, s, w.gccnt, w.g_size,
                       w.rscan, w.rscan + kClasses, w.glist, w.counters);
}

}  // namespace hf
