// L0 friends-of-friends over the particles denser than Delta_L0,min (Sec. 2.2.1):
// two members are friends when their separation is less than l; L0 groups are
// the connected components.
//
// Lock-free union-find in sorted (cell, sub-cell) order:
//   phase A  a sub-cell's diagonal is below l, so all members of a sub-cell are
//            friends: in dense cells every member points at the first member of
//            its sub-cell;
//   cells    a head start for the dense cells: sub-cells next to each other
//            whose first members are friends are joined, inside a cell without
//            atomics, then across cell faces; a cell whose members are all in
//            one set then carries that set's root;
//   dense    one wavefront per dense chunk gathers the neighbour members within
//            reach 64 at a time and tests them against its lanes (FP32
//            prefilter on the cell-local coordinates, canonical FP64 distance
//            for the undecided band); it joins sets in its own view of the
//            forest and applies the resulting hooks in bulk;
//   sparse   members of sparse cells link to the members of sparse neighbour
//            cells in the forward half of the stencil;
//   labels   compression, then 1 + the smallest ORIGINAL index of each set.
// Hooks always attach the larger root under the smaller one, so the sets, and
// therefore the labels, do not depend on thread scheduling.
#include "hf_internal.h"

namespace hf {

namespace {

inline dim3 grid(int64_t n) { return dim3((unsigned)((n + kBlock - 1) / kBlock)); }

__device__ __forceinline__ int ld(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st(int32_t *p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root with path halving.  Only non-roots are rewritten and only ever to an
// ancestor, so the relaxed stores cannot undo a concurrent hook (hooks only
// change roots).
__device__ int uf_find(int32_t *parent, int x) {
    for (;;) {
        int p = ld(parent + x);
        if (p == x) return x;
        int gp = ld(parent + p);
        if (gp != p) st(parent + x, gp);
        x = gp;
    }
}

// Root by plain (cacheable) loads, for filters only: a stale parent is an
// earlier ancestor, so two particles reported in one set are in one set; a
// "different" answer may be stale and is then settled by uf_unite.
__device__ __forceinline__ int uf_find_hint(const int32_t *parent, int x) {
    for (;;) {
        const int p = parent[x];
        if (p == x) return x;
        x = p;
    }
}

// The same once parent p of x is known.
__device__ __forceinline__ int uf_find_from(const int32_t *parent, int x, int p) {
    return p == x ? x : uf_find_hint(parent, p);
}

__device__ void uf_unite(int32_t *parent, int a, int b) {
    for (;;) {
        a = uf_find(parent, a);
        b = uf_find(parent, b);
        if (a == b) return;
        if (a > b) { int t = a; a = b; b = t; }
        int old = atomicCAS(parent + b, b, a);
        if (old == b) return;
    }
}

// Hooks a wavefront has decided on but not yet applied to the forest: lane
// k < n holds hook k, a root c to be attached under p < c.  Deferring them
// takes the compare-and-swap round trips out of the serial candidate loop:
// the wavefront joins sets in its own registers and applies all hooks at
// once, one lane each.
struct Hooks {
    int c = -1, p = -1, n = 0;
};

// Applies every queued hook: a compare-and-swap while c is still a root,
// otherwise a full union (c was hooked elsewhere meanwhile).
__device__ __forceinline__ void hooks_apply(int32_t *parent, Hooks &h) {
    if ((int)(threadIdx.x & 63) < h.n && atomicCAS(parent + h.c, h.c, h.p) != h.c) uf_unite(parent, h.c, h.p);
    h.n = 0;
}

__device__ __forceinline__ void hooks_push(int32_t *parent, Hooks &h, int c, int p) {
    if (h.n == 64) hooks_apply(parent, h);
    if ((int)(threadIdx.x & 63) == h.n) {
        h.c = c;
        h.p = p;
    }
    h.n++;
}

// A root hint read from the forest, moved through the queued hooks in the
// order they were queued: a hook's parent was a root of the wavefront's view
// when queued, so only a later hook can move it again.
__device__ __forceinline__ int hooks_map(const Hooks &h, int x) {
    for (int k = 0; k < h.n; k++)
        if (x == lane_get(h.c, k)) x = lane_get(h.p, k);
    return x;
}

// The lanes lk are linked to a particle whose set has the local root r.  In
// the wavefront's view of the forest (every root it holds is a node of its
// set), the smallest of r and the lanes' roots becomes the root of all of
// them; the others are queued as hooks under it, and every reference the
// wavefront holds to one of them (lane roots wr, candidate roots rc, task
// roots rt) is moved to it.
__device__ __forceinline__ void join_local(int32_t *parent, Hooks &h, bool lk, int r, int &wr, int &rc, int &rt) {
    // the smallest root: one step per distinct root among the linked lanes
    // (rarely more than one or two), with no cross-lane shuffle
    int m = r;
    for (uint64_t mask = __ballot(lk); mask;) {
        const int x = lane_get(wr, (int)__builtin_ctzll(mask));
        m = min(m, x);
        mask &= ~__ballot(wr == x);
    }
    if (r != m) {
        hooks_push(parent, h, r, m);
        if (wr == r) wr = m;
        if (rc == r) rc = m;
        if (rt == r) rt = m;
    }
    uint64_t mask;
    while ((mask = __ballot(lk && wr != m)) != 0ull) {
        const int x = lane_get(wr, (int)__builtin_ctzll(mask));
        hooks_push(parent, h, x, m);
        if (wr == x) wr = m;
        if (rc == x) rc = m;
        if (rt == x) rt = m;
    }
}

// Tests the member candidates of a batch (lane p: candidate p) against the
// chunk's lanes and joins their sets.  A candidate holds whether it is a
// member, its coordinates in the chunk's cell frame (units of b), its index
// and its local root rc; a candidate already in the set of every lane needs no
// test.  The loop runs over the smaller side: with fewer candidates than chunk
// particles, each candidate is broadcast to the chunk's lanes and joined to
// the lanes it links at once; otherwise the candidates stay in the lanes, the
// chunk's particles are broadcast one after the other (each candidate
// collecting a bit mask of the lanes it links), and the linked candidates are
// joined one after the other.
__device__ __forceinline__ void test_candidates(int32_t *parent, Hooks &h, const float4 *__restrict__ spos,
                                                const Geo &g, bool active, const float4 &li, uint32_t h0,
                                                int &wr, bool cmem, float qx, float qy, float qz, uint32_t cj,
                                                int &rc, int &rt) {
    const int lane = threadIdx.x & 63;
    const uint64_t am = __ballot(active);
    const int w0 = lane_get(wr, (int)__builtin_ctzll(am));
    const bool common = !__ballot(active && wr != w0);
    const bool need = cmem && !(common && rc == w0);
    const uint64_t nm = __ballot(need);
    if (!nm) return;
    if (__popcll(nm) < __popcll(am)) {
        for (uint64_t mm = nm; mm; mm &= mm - 1) {
            const int J = (int)__builtin_ctzll(mm);
            const int r = lane_get(rc, J);
            if (!__ballot(active && wr != r)) continue;
            const float dx = lane_get(qx, J) - li.x, dy = lane_get(qy, J) - li.y, dz = lane_get(qz, J) - li.z;
            const float d2f = d2_f32(dx, dy, dz);
            bool lk = active && wr != r && d2f < g.l2b_hi;
            if (lk && !(d2f < g.l2b_lo)) lk = d2_exact(spos[h0 + (uint32_t)lane], spos[lane_get(cj, J)], g.L, g.half) < g.l2;
            if (__ballot(lk)) join_local(parent, h, lk, r, wr, rc, rt);
        }
        return;
    }
    uint32_t lo = 0u, hi = 0u;  // linked chunk lanes 0..31 and 32..63
    for (uint64_t m = am; m; m &= m - 1) {
        const int I = (int)__builtin_ctzll(m);
        const float dx = qx - lane_get(li.x, I), dy = qy - lane_get(li.y, I), dz = qz - lane_get(li.z, I);
        const float d2f = d2_f32(dx, dy, dz);
        bool lk = need && d2f < g.l2b_hi;
        if (lk && !(d2f < g.l2b_lo)) lk = d2_exact(spos[h0 + (uint32_t)I], spos[cj], g.L, g.half) < g.l2;
        if (I < 32)
            lo |= lk ? 1u << I : 0u;
        else
            hi |= lk ? 1u << (I - 32) : 0u;
    }
    for (uint64_t mm = __ballot((lo | hi) != 0u); mm; mm &= mm - 1) {
        const int J = (int)__builtin_ctzll(mm);
        const int r = lane_get(rc, J);
        const uint32_t bits = lane < 32 ? lane_get(lo, J) >> lane : lane_get(hi, J) >> (lane - 32);
        const bool lk = (bits & 1u) != 0u && wr != r;
        if (__ballot(lk)) join_local(parent, h, lk, r, wr, rc, rt);
    }
}

// Phase A, which also initializes the forest: non-members get -1, members of
// sparse cells are roots, and members of dense cells point at the first member
// of their sub-cell (a valid forest: every parent is a member with a smaller
// or equal sorted index).  The first particle of every dense sub-cell also
// records the sub-cell's first member (-1 if none) in submem, laid out like
// the sub-cell table.  The smallest index of every set that starts here (no
// other particle becomes a root) and the member counts start here too, and the
// members of sparse cells (about one in ten of their particles) are listed.
template <int kPhaseAPer>  // particles per thread
__global__ __launch_bounds__(kBlock) void k_fof_phase_a(int64_t n, Boxes bx, Marks marks,
                                                        const uint16_t *__restrict__ ssub,
                                                        const uint32_t *__restrict__ subtab,
                                                        const float *__restrict__ dens_s,
                                                        int32_t *__restrict__ parent,
                                                        int32_t *__restrict__ submem,
                                                        int32_t *__restrict__ minorig,
                                                        uint32_t *__restrict__ gcnt, SegList sl,
                                                        uint64_t *clock) {
    stamp(clock);
    const int64_t i0 = (int64_t)xcd_block() * (kPhaseAPer * kBlock) + threadIdx.x;
    int si[kPhaseAPer];
    uint32_t cell[kPhaseAPer], u0[kPhaseAPer];
    bool mem[kPhaseAPer], sp[kPhaseAPer], listed[kPhaseAPer];
    int32_t idx[kPhaseAPer];
    // everything indexed by i in one round of loads
#pragma unroll
    for (int u = 0; u < kPhaseAPer; u++) {
        const int64_t i = i0 + u * kBlock, ic = i < n ? i : n - 1;
        si[u] = ssub[ic];
        cell[u] = dense_ordinal(marks, (uint32_t)ic);
        mem[u] = i < n && is_member(dens_s, ic, bx.geo[box_of(bx, (uint32_t)ic)].dl0);
        sp[u] = i >= n || is_sparse(marks, ic);
        listed[u] = i < n && sp[u] && mem[u];
        idx[u] = (int32_t)i;
    }
#pragma unroll
    for (int u = 0; u < kPhaseAPer; u++) u0[u] = sp[u] ? 0u : subtab[(int64_t)cell[u] * (bx.nsub_max + 1) + si[u]];
    seg_append<kPhaseAPer>(sl, listed, idx);
#pragma unroll
    for (int u = 0; u < kPhaseAPer; u++) {
        const int64_t i = i0 + u * kBlock;
        if (i >= n) break;
        gcnt[i] = 0u;
        if (sp[u]) {
            parent[i] = mem[u] ? (int32_t)i : -1;
            if (mem[u]) minorig[i] = 0x7fffffff;
            continue;
        }
        const double dl0 = bx.geo[box_of(bx, (uint32_t)i)].dl0;
        if (mem[u]) {
            uint32_t f = u0[u];
            while (f < (uint32_t)i && !is_member(dens_s, f, dl0)) f++;
            parent[i] = (int32_t)f;
            if (f == (uint32_t)i) minorig[i] = 0x7fffffff;
        } else {
            parent[i] = -1;
        }
        if ((uint32_t)i == u0[u]) {
            const int64_t row = (int64_t)cell[u] * (bx.nsub_max + 1) + si[u];
            const uint32_t u1 = subtab[row + 1];
            uint32_t f = u0[u];
            while (f < u1 && !is_member(dens_s, f, dl0)) f++;
            submem[row] = f < u1 ? (int32_t)f : -1;
        }
    }
}

// ------------------------------------------------------------ dense cells
// The chunk kernel below starts from a forest in which every sub-cell is a set
// of its own, and all chunks run at once: on a small box each of them tested
// its whole neighbourhood before another one's joins could save it the work
// (99 us on the 64^3 box, the longest chunk's chain), and on a large one two
// thirds of the tests joined what a neighbour had joined meanwhile (1.72 ms on
// the 256^3 box, 22.4 ms on the 512^3 one).  Three short kernels make the links
// that cost next to nothing to find: between the first members of sub-cells that
// touch.

// The first member of the sub-cell in this row of the table, -1 for none
// (phase A writes submem for sub-cells that hold particles only).
__device__ __forceinline__ int32_t sub_first(const uint32_t *__restrict__ subtab,
                                             const int32_t *__restrict__ submem, int64_t row) {
    const uint32_t u0 = subtab[row], u1 = subtab[row + 1];
    const int32_t f = submem[row];
    return u1 > u0 ? f : -1;
}

// Inside a cell, half a wavefront per cell, a lane per sub-cell: every sub-cell
// is attached to the first of the sub-cells before it that touch it and whose
// first member is a friend of its own (13 offsets).  Parents come earlier in
// the order, so this is a forest, and nothing else touches the roots of this
// cell's sub-cells yet: plain stores.  Sub-cells of one set may be left in two
// trees here, which the later kernels join.  (Exact components by a search on
// 64-bit link masks, a wavefront per cell, took 234 us on the 256^3 box, bound
// by the scalar unit.)
constexpr int kHalves = kBlock / 32;
__global__ __launch_bounds__(kBlock) void k_fof_cells(int64_t ndc, Boxes bx,
                                                      const float4 *__restrict__ sloc,
                                                      const uint32_t *__restrict__ subtab,
                                                      const int32_t *__restrict__ submem,
                                                      int32_t *__restrict__ parent) {
    extern __shared__ float4 s_first[];  // [kHalves][nsub_max]: first member's position, its index in w
    const int hw = threadIdx.x >> 5, ln = threadIdx.x & 31;
    const int64_t d = (int64_t)xcd_block() * kHalves + hw;
    if (d >= ndc) return;
    float4 *sp = s_first + hw * bx.nsub_max;
    const int64_t row = d * (bx.nsub_max + 1);
    per_box(bx, box_of(bx, subtab[row]), [&](const Geo &g) {
    const int k = g.ksub, nsub = g.nsub;
    for (int s = ln; s < nsub; s += 32) {
        const int32_t fm = sub_first(subtab, submem, row + s);
        float4 p = make_float4(1e8f, 0.0f, 0.0f, 0.0f);  // empty: far from everything
        if (fm >= 0) p = sloc[fm];
        p.w = __int_as_float(fm);
        sp[s] = p;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
    const float inv_k = 1.0f / (float)k, inv_k2 = 1.0f / (float)(k * k);
    for (int s = ln; s < nsub; s += 32) {
        const float4 p = sp[s];
        const int32_t fm = __float_as_int(p.w);
        if (fm < 0) continue;
        const int sz = div_small(s, inv_k2), syx = s - sz * k * k, sy = div_small(syx, inv_k), sx = syx - sy * k;
        int32_t to = fm;
#pragma unroll
        for (int e = 0; e < 13; e++) {
            // backward offsets: stencil indices 0..12
            const int dx = e % 3 - 1, dy = (e / 3) % 3 - 1, dz = e / 9 - 1;
            const bool ok = sx + dx >= 0 && sx + dx < k && sy + dy >= 0 && sy + dy < k && sz + dz >= 0;
            const float4 q = sp[ok ? s + (dz * k + dy) * k + dx : s];
            if (ok && d2_f32(q.x - p.x, q.y - p.y, q.z - p.z) < g.l2b_lo) to = min(to, __float_as_int(q.w));
        }
        if (to != fm) parent[fm] = to;
    }
    });
}

// Across cells, half a wavefront per cell: the pairs of sub-cells that touch
// through the cell's three forward faces, one per lane (27 for k = 3).  Of the
// pairs that would join the same two sets one lane joins them.
__global__ __launch_bounds__(kBlock) void k_fof_faces(int64_t ndc, Boxes bx,
                                                      const uint32_t *__restrict__ dcells,
                                                      Cells cells, const float4 *__restrict__ sloc,
                                                      const uint32_t *__restrict__ subtab,
                                                      const int32_t *__restrict__ submem,
                                                      int32_t *parent) {
    const int hw = threadIdx.x >> 5, ln = threadIdx.x & 31, hsh = threadIdx.x & 32;
    const int64_t d = (int64_t)xcd_block() * kHalves + hw;
    if (d >= ndc) return;
    auto hballot = [&](bool p) { return (uint32_t)(__ballot(p) >> hsh); };
    const uint32_t c = dcells[d];
    const int tstride = bx.nsub_max + 1;
    per_box(bx, box_of(bx, subtab[d * tstride]), [&](const Geo &g) {
    const int k = g.ksub, k2 = k * k;
    const float inv_k = 1.0f / (float)k, inv_k2 = 1.0f / (float)k2;
    int cx, cy, cz;
    cell_xyz(g, c, cx, cy, cz);
    for (int t0 = 0; t0 < 3 * k2; t0 += 32) {
        const int t = t0 + ln;
        int32_t r1 = -1, r2 = -1;
        if (t < 3 * k2) {
            const int ax = div_small(t, inv_k2), r = t - ax * k2, v = div_small(r, inv_k), u = r - v * k;
            const uint32_t nb = cell_id(g, cx + (ax == 0), cy + (ax == 1), cz + (ax == 2));
            uint32_t na, ne;
            const uint32_t o = cell_range(cells, nb, na, ne);
            if (ne - na >= (uint32_t)kDenseMin) {
                // the last layer of sub-cells here, the first one there
                const int st = ax == 0 ? 1 : (ax == 1 ? k : k2);
                const int s2 = ax == 0 ? v * k2 + u * k : (ax == 1 ? v * k2 + u : v * k + u);
                const int32_t f1 = sub_first(subtab, submem, d * tstride + s2 + (k - 1) * st);
                const int32_t f2 = sub_first(subtab, submem, (int64_t)cells.dmap[o] * tstride + s2);
                if (f1 >= 0 && f2 >= 0) {
                    const float4 p = sloc[f1], q = sloc[f2];
                    const float dx = q.x + (ax == 0 ? g.cellb : 0.0f) - p.x,
                                dy = q.y + (ax == 1 ? g.cellb : 0.0f) - p.y,
                                dz = q.z + (ax == 2 ? g.cellb : 0.0f) - p.z;
                    if (d2_f32(dx, dy, dz) < g.l2b_lo) {
                        r1 = uf_find_hint(parent, f1);
                        r2 = uf_find_hint(parent, f2);
                    }
                }
            }
        }
        bool join = false;
        for (uint32_t m = hballot(r1 != r2); m;) {
            const int L = __ffs(m) - 1;
            const int x = __shfl(r1, L, 32), y = __shfl(r2, L, 32);
            if (ln == L) join = true;
            m &= ~hballot(r1 == x && r2 == y);
        }
        if (join) uf_unite(parent, r1, r2);
    }
    });
}

// The first members' roots, stored as their parents (the forest does not
// change here), and per cell, in entry nsub_max of its row: the root when all
// its members are in one set, -1 when they are not, -2 when it has none.
__global__ __launch_bounds__(kBlock) void k_fof_cell_roots(int64_t ndc, Boxes bx,
                                                           const uint32_t *__restrict__ subtab,
                                                           int32_t *__restrict__ submem, int32_t *parent) {
    const int hw = threadIdx.x >> 5, ln = threadIdx.x & 31, hsh = threadIdx.x & 32;
    const int64_t d = (int64_t)xcd_block() * kHalves + hw;
    if (d >= ndc) return;
    int nsub = 0;
    const int64_t row = d * (bx.nsub_max + 1);
    per_box(bx, box_of(bx, subtab[row]), [&](const Geo &g) { nsub = g.nsub; });
    int32_t one = -2;
    for (int s0 = 0; s0 < nsub; s0 += 32) {
        const int32_t fm = s0 + ln < nsub ? sub_first(subtab, submem, row + s0 + ln) : -1;
        int32_t r = -1;
        if (fm >= 0) {
            r = fm;
            for (int p = ld(parent + r); p != r; p = ld(parent + r)) r = p;
            st(parent + fm, r);
        }
        const uint32_t m = (uint32_t)(__ballot(fm >= 0) >> hsh);
        if (!m) continue;
        const int32_t f = __shfl(r, __ffs(m) - 1, 32);
        const bool split = (uint32_t)(__ballot(fm >= 0 && r != f) >> hsh) != 0u;
        one = split || (one != -2 && one != f) ? -1 : f;
    }
    if (ln == 0) submem[row + bx.nsub_max] = one;
}

// Sub-cells examined at a time by the dense kernel.
constexpr int kTaskTile = 384;

// Dense chunks, one wavefront each (lanes = the chunk's particles).  The wave
// visits the neighbour cells that come within l of some lane: sparse cells in
// all 26 directions, dense cells only in the forward half (the backward ones
// visit this cell themselves), and its own cell from the chunk start on.
// The 27 cell ranges are loaded at once (one stencil cell per lane).
// Neighbour particles are gathered 64 at a time (one per lane, shifted into
// the chunk's cell frame) and tested one after the other against all lanes;
// sets are joined in the wavefront's registers and the hooks applied to the
// forest in bulk before each round of sub-cells and at the end (root hints read
// meanwhile are moved through the queued hooks; applying them and reading the
// roots again after every gather round with joins was a chain of round trips
// for little: 852 us on the 256^3 box, 815 without, 795 gathering 64 instead of
// 32 at a time):
//   sparse cells  all their particles, each member with its root;
//   dense cells   their sub-cells, kTaskTile at a time: range and first member
//                 (recorded by phase A); those with members within reach are
//                 listed in LDS and taken 64 at a time (one per lane) with
//                 that member's root.  A sub-cell already in the set of every
//                 lane is passed over (its members are one set); the
//                 particles of the others are gathered in lane order.  (Most
//                 of the up to 378 sub-cells are empty or out of reach: taken
//                 64 at a time unlisted, each round refreshed the forest and
//                 the roots for a few of them.)
// A dense cell that carries the root common to all lanes has nothing to join
// and is not visited.
// With nparts > 1 a chunk is a wavefront for the sparse cells and nparts - 1 for
// the sub-cells of the dense ones: for inputs whose chunks do not fill the chip,
// where the longest chain is the time.
__global__ __launch_bounds__(64, 8) void k_fof_dense(int64_t nchunks, unsigned tile, int nparts, int64_t n, Boxes bx,
                                                      const int32_t *__restrict__ chunks,
                                                      const float4 *__restrict__ sloc,
                                                      const float4 *__restrict__ spos,
                                                      Cells cells, Marks marks,
                                                      const uint32_t *__restrict__ subtab,
                                                      const int32_t *__restrict__ submem,
                                                      const float *__restrict__ dens_s,
                                                      int32_t *parent) {
    __shared__ int64_t dbase[27];  // visited dense cells: sub-table base
    __shared__ int8_t doff[27];    // and stencil index
    __shared__ int32_t s_fs[kTaskTile];   // sub-cells to look at: first member to gather,
    __shared__ uint32_t s_u1[kTaskTile];  // end,
    __shared__ int8_t s_st[kTaskTile];    // stencil index
    const unsigned wq = xcd_tile_block(tile);
    const int64_t q = wq / (unsigned)nparts;
    if (q >= nchunks) return;
    // wavefront 0 of several takes the sparse cells, the others every
    // shares-th sub-cell of each dense one (which cells a wavefront visits
    // depends on the joins it sees, so the shares are cut within the cells)
    const int role = (int)(wq - (unsigned)q * (unsigned)nparts), shares = max(nparts - 1, 1), share = max(role - 1, 0);
    const bool do_sparse = role == 0, do_dense = nparts == 1 || role > 0;
    const int lane = threadIdx.x & 63;
    const uint32_t h = (uint32_t)__builtin_amdgcn_readfirstlane(chunks[q]);
    const Geo &g = bx.geo[__builtin_amdgcn_readfirstlane(box_of(bx, h))];
    const uint32_t c = __builtin_amdgcn_readfirstlane(__float_as_uint(sloc[h].w));
    const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane(chunk_end(marks, h, n));
    const uint32_t i = h + (uint32_t)lane;
    const uint32_t ic = i < end ? i : h;
    // a particle is a member if it has a parent
    const int up = parent[ic];
    const bool active = i < end && up >= 0;
    if (!__ballot(active)) return;
    const float4 li = sloc[ic];
    int wr = active ? uf_find_from(parent, (int)ic, up) : -1;
    const int k = g.ksub, nsub = g.nsub, tstride = bx.nsub_max + 1;
    const float subb = g.cellb / (float)k;
    int cx, cy, cz;
    cell_xyz(g, c, cx, cy, cz);
    // one stencil cell per lane (offset (t % 3 - 1, t / 3 % 3 - 1, t / 9 - 1)):
    // its index word here, its range below if it comes within l of the chunk's box
    const int tl = lane < 27 ? lane : 13;
    const int lx = tl % 3 - 1, ly = (tl / 3) % 3 - 1, lz = tl / 9 - 1;
    const uint32_t nbl = cell_id(g, cx + lx, cy + ly, cz + lz);
    const uint2 nbw = cells.occ[nbl / kOccCells];
    // chunk bounding box (active lanes), for the reach tests of stencil cells
    // and sub-cells
    float bx0 = active ? li.x : 1e30f, by0 = active ? li.y : 1e30f, bz0 = active ? li.z : 1e30f;
    float bx1 = active ? li.x : -1e30f, by1 = active ? li.y : -1e30f, bz1 = active ? li.z : -1e30f;
    bx0 = wave_min(bx0);
    by0 = wave_min(by0);
    bz0 = wave_min(bz0);
    bx1 = wave_max(bx1);
    by1 = wave_max(by1);
    bz1 = wave_max(bz1);
    const float gx = lx < 0 ? bx0 : (lx > 0 ? g.cellb - bx1 : 0.0f);
    const float gy = ly < 0 ? by0 : (ly > 0 ? g.cellb - by1 : 0.0f);
    const float gz = lz < 0 ? bz0 : (lz > 0 ? g.cellb - bz1 : 0.0f);
    const bool lreach = lane < 27 && gx * gx + gy * gy + gz * gz < g.l2b_hi;
    uint32_t la = 0, lb = 0, lo = 0;
    if (lreach) lo = cell_range(cells, nbw, nbl, la, lb);
    const bool ldense = lb - la >= (uint32_t)kDenseMin;
    const bool lforward = lz > 0 || (lz == 0 && (ly > 0 || (ly == 0 && lx >= 0)));  // own cell included
    const int wfirst = lane_get(wr, (int)__builtin_ctzll(__ballot(active)));
    const bool wsame = !__ballot(active && wr != wfirst);
    bool lvisit = do_dense && lreach && ldense && lforward;
    int64_t lbase = 0;
    if (lvisit) {
        lbase = (int64_t)cells.dmap[lo] * tstride;
        const int32_t cr = submem[lbase + bx.nsub_max];
        lvisit = cr != -2 && !(wsame && cr == wfirst);
    }
    if (lvisit) {
        const uint64_t vm = __ballot(lvisit);
        const int slot = __popcll(vm & ((1ull << lane) - 1ull));
        dbase[slot] = lbase;
        doff[slot] = (int8_t)lane;
    }
    const int nvisit = __popcll(__ballot(lvisit));
    Hooks hk;
    int no_rt = -1;
    // sparse neighbour cells: their particles numbered through a prefix sum of
    // the cell sizes; lane p finds the cell of particle p by one walk over the
    // cells that hold particles (their starts are scalars)
    {
        const int cntl = do_sparse && lreach && !ldense ? (int)(lb - la) : 0;
        const int incl = (int)wave_incl_scan((uint32_t)cntl);
        const int P = lane_get(incl, 63);
        const uint64_t cells = __ballot(cntl > 0);
        for (int p0 = 0; p0 < P; p0 += 64) {
            const int p = p0 + lane;
            int t = 0;
            uint32_t jt = 0;
            for (uint64_t m = cells; m; m &= m - 1) {
                const int u = (int)__builtin_ctzll(m);
                const int stt = lane_get(incl, u) - lane_get(cntl, u);
                if (p >= stt) {
                    t = u;
                    jt = lane_get(la, u) + (uint32_t)(p - stt);
                }
            }
            bool cmem = false;
            float qx = 0.0f, qy = 0.0f, qz = 0.0f;
            int rc = -1;
            if (p < P) {
                const float4 lj = sloc[jt];
                const int upj = parent[jt];
                cmem = upj >= 0;
                rc = upj;
                qx = lj.x + (float)(t % 3 - 1) * g.cellb;
                qy = lj.y + (float)((t / 3) % 3 - 1) * g.cellb;
                qz = lj.z + (float)(t / 9 - 1) * g.cellb;
            }
            if (cmem) rc = hooks_map(hk, uf_find_from(parent, (int)jt, rc));
            test_candidates(parent, hk, spos, g, active, li, h, wr, cmem, qx, qy, qz, jt, rc, no_rt);
        }
    }
    if (nvisit > 0) {
        __builtin_amdgcn_wave_barrier();
        const int a0 = (int)__builtin_ctzll(__ballot(active));
        const int nmine = (nsub - share + shares - 1) / shares;  // sub-cells of this share per cell
        const int ntask = nvisit * nmine;
        const float inv_mine = 1.0f / (float)nmine, inv_k = 1.0f / (float)k, inv_k2 = 1.0f / (float)(k * k);
        for (int tb = 0; tb < ntask; tb += kTaskTile) {
        int listed = 0;
        constexpr int kTb = 3;  // 64-task rounds whose loads are issued together
        for (int r0 = tb; r0 < tb + kTaskTile && r0 < ntask; r0 += 64 * kTb) {
            uint32_t u0[kTb], u1[kTb];
            int32_t fm[kTb];
            int stv[kTb], sl[kTb];
#pragma unroll
            for (int r = 0; r < kTb; r++) {
                const int tq = r0 + 64 * r + lane;
                u0[r] = u1[r] = 0u;
                fm[r] = -1;
                stv[r] = sl[r] = 0;
                if (tq < ntask) {
                    const int cell = div_small(tq, inv_mine);
                    sl[r] = (tq - cell * nmine) * shares + share;
                    stv[r] = doff[cell];
                    const int64_t row = dbase[cell] + sl[r];
                    u0[r] = subtab[row];
                    u1[r] = subtab[row + 1];
                    fm[r] = submem[row];
                }
            }
#pragma unroll
            for (int r = 0; r < kTb; r++) {
                int fs = -1;
                if (u1[r] > u0[r]) {
                    const bool cut = stv[r] == 13 && u0[r] < h;  // own cell: from the chunk start on
                    const int ox = stv[r] % 3 - 1, oy = (stv[r] / 3) % 3 - 1, oz = stv[r] / 9 - 1;
                    const int sz = div_small(sl[r], inv_k2), syx = sl[r] - sz * k * k, sy = div_small(syx, inv_k),
                              sx = syx - sy * k;
                    // sub-cell box (neighbour frame) shifted into the chunk's frame
                    const float ex = fmaxf(fmaxf(sx * subb + (float)ox * g.cellb - bx1,
                                                 bx0 - ((sx + 1) * subb + (float)ox * g.cellb)), 0.0f);
                    const float ey = fmaxf(fmaxf(sy * subb + (float)oy * g.cellb - by1,
                                                 by0 - ((sy + 1) * subb + (float)oy * g.cellb)), 0.0f);
                    const float ez = fmaxf(fmaxf(sz * subb + (float)oz * g.cellb - bz1,
                                                 bz0 - ((sz + 1) * subb + (float)oz * g.cellb)), 0.0f);
                    if (ex * ex + ey * ey + ez * ez < g.l2b_hi + 1e-4f) {
                        // first member: recorded by phase A, searched where the
                        // own cell's sub-cell is cut at the chunk start
                        if (!cut) {
                            fs = fm[r];
                        } else {
                            for (uint32_t j = h; j < u1[r]; j++)
                                if (is_member(dens_s, j, g.dl0)) {
                                    fs = (int)j;
                                    break;
                                }
                        }
                    }
                }
                const uint64_t km = __ballot(fs >= 0);
                if (fs >= 0) {
                    const int at = listed + __popcll(km & ((1ull << lane) - 1ull));
                    s_fs[at] = fs;
                    s_u1[at] = u1[r];
                    s_st[at] = (int8_t)stv[r];
                }
                listed += __popcll(km);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        // the listed sub-cells, 64 at a time
        for (int t0 = 0; t0 < listed; t0 += 64) {
            // the forest learns this chunk's joins so far, the lanes their
            // current roots (a sub-cell joined meanwhile, by any chunk, is
            // then passed over)
            hooks_apply(parent, hk);
            if (active) wr = uf_find_hint(parent, wr);
            const bool has = t0 + lane < listed;
            const int fs = has ? s_fs[t0 + lane] : -1, st = has ? (int)s_st[t0 + lane] : 0;
            const uint32_t u1 = has ? s_u1[t0 + lane] : 0u;
            int rt = fs >= 0 ? hooks_map(hk, uf_find_hint(parent, fs)) : -1;
            uint32_t pos = fs >= 0 ? (uint32_t)fs : 0u;  // next particle of the sub-cell to gather
            for (;;) {
                const int w0 = lane_get(wr, a0);
                const int wcommon = __ballot(active && wr != w0) ? -2 : w0;
                const uint32_t len = fs >= 0 && pos < u1 && rt != wcommon ? u1 - pos : 0u;
                const uint32_t incl = wave_incl_scan(len);
                const uint32_t T = lane_get(incl, 63);
                if (T == 0) break;
                // lane p takes particle p of the sub-cells' runs laid end to end
                int tst = 13, trt = -1;
                uint32_t jt = 0;
                for (uint64_t m = __ballot(len > 0); m; m &= m - 1) {
                    const int u = (int)__builtin_ctzll(m);
                    const uint32_t stu = lane_get(incl, u) - lane_get(len, u);
                    if (stu >= 64u) break;
                    if ((uint32_t)lane >= stu) {
                        tst = lane_get(st, u);
                        trt = lane_get(rt, u);
                        jt = lane_get(pos, u) + ((uint32_t)lane - stu);
                    }
                }
                // every sub-cell moves past what this round takes from it
                const uint32_t mine = incl - len;
                if (mine < 64u) pos += min(len, 64u - mine);
                bool cmem = false;
                float qx = 0.0f, qy = 0.0f, qz = 0.0f;
                int rc = -1;
                if ((uint32_t)lane < T) {
                    const float4 lj = sloc[jt];
                    cmem = is_member(dens_s, jt, g.dl0);
                    qx = lj.x + (float)(tst % 3 - 1) * g.cellb;
                    qy = lj.y + (float)((tst / 3) % 3 - 1) * g.cellb;
                    qz = lj.z + (float)(tst / 9 - 1) * g.cellb;
                    rc = trt;
                }
                test_candidates(parent, hk, spos, g, active, li, h, wr, cmem, qx, qy, qz, jt, rc, rt);
            }
        }
        __builtin_amdgcn_wave_barrier();
        }
    }
    hooks_apply(parent, hk);
}

// Members of sparse cells (listed by phase A): links to the members of the
// sparse cells in the forward half of the stencil (own cell: the later ones),
// so each pair is seen once; pairs with dense cells are found by the dense
// chunks.  Sixteen lanes per member, one stencil cell each (14 of them): the
// ranges, then all densities and positions of a cell (seven at most) are one
// round of loads each.  The links (two or three per member) are queued in LDS
// and joined 64 at a time, one per lane: a join is a chain of its own, and
// joined where they were found the links of a lane ran one after the other
// with most lanes idle (925 us on the 256^3 box).  One thread per member, the
// 27 cells walked as a chain of dependent loads, took 76 us on the 64^3 box and
// 333 us on the 256^3 one, with 20 us of flags, scan and list before it.
constexpr int kLinkMost = (64 / 16) * 14 * (kDenseMin - 1);  // links of a round of a wavefront
__global__ __launch_bounds__(kBlock, 8) void k_fof_sparse(SegList sl, Boxes bx,
                                                       const float4 *__restrict__ sloc,
                                                       const float4 *__restrict__ spos,
                                                       Cells cells, const float *__restrict__ dens_s,
                                                       int32_t *parent) {
    __shared__ int2 s_link[kBlock / 64][64 + kLinkMost];
    __shared__ uint32_t s_n[kBlock / 64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, ln = threadIdx.x & 15;
    // the forward half: stencil cells 13 (own) .. 26
    const int ox = (ln + 13) % 3 - 1, oy = ((ln + 13) / 3) % 3 - 1, oz = (ln + 13) / 9 - 1;
    const SegShare sh = seg_share<16>(sl);
    uint32_t queued = 0;
    auto join = [&](uint32_t cnt) {
        queued -= cnt;
        if ((uint32_t)lane < cnt) {
            const int2 l = s_link[w][queued + (uint32_t)lane];
            // most links are inside a set by now: plain loads tell
            const int x = uf_find_hint(parent, l.x), y = uf_find_hint(parent, l.y);
            if (x != y) uf_unite(parent, x, y);
        }
    };
    for (uint32_t k = sh.k; __ballot(k < sh.n) != 0ull; k += sh.step) {
        uint32_t links = 0, a = 0;
        int i = 0;
        if (k < sh.n && ln < 14) {
            i = sl.list[(int64_t)sh.seg * sl.cap + k];
            const float4 li = sloc[i];
            per_box(bx, box_of(bx, (uint32_t)i), [&](const Geo &g) {
            const float gx = ox < 0 ? li.x : (ox > 0 ? g.cellb - li.x : 0.0f);
            const float gy = oy < 0 ? li.y : (oy > 0 ? g.cellb - li.y : 0.0f);
            const float gz = oz > 0 ? g.cellb - li.z : 0.0f;
            if (gx * gx + gy * gy + gz * gz < g.l2b_hi) {
                int cx, cy, cz;
                cell_xyz(g, __float_as_uint(li.w), cx, cy, cz);
                const uint32_t nb = cell_id(g, cx + ox, cy + oy, cz + oz);
                uint32_t b;
                cell_range(cells, nb, a, b);
                if (b - a >= (uint32_t)kDenseMin) b = a;
                if (ln == 0) a = (uint32_t)i + 1u;
                const float xs = li.x - (float)ox * g.cellb, ys = li.y - (float)oy * g.cellb,
                            zs = li.z - (float)oz * g.cellb;
                float dj[kDenseMin - 1];
                float3 lj[kDenseMin - 1];
#pragma unroll
                for (uint32_t v = 0; v < kDenseMin - 1; v++) {
                    const float *const p = reinterpret_cast<const float *>(sloc + (a + v));
                    dj[v] = 0.0f;
                    lj[v] = make_float3(0.0f, 0.0f, 0.0f);
                    if (a + v < b) {
                        dj[v] = dens_s[a + v];
                        lj[v] = make_float3(p[0], p[1], p[2]);
                    }
                }
                uint32_t open = 0;
#pragma unroll
                for (uint32_t v = 0; v < kDenseMin - 1; v++) {
                    const float d2f = d2_f32(lj[v].x - xs, lj[v].y - ys, lj[v].z - zs);
                    const bool near = a + v < b && (double)dj[v] > g.dl0 && d2f < g.l2b_hi;
                    if (near) (d2f < g.l2b_lo ? links : open) |= 1u << v;
                }
                // the undecided band, by the canonical distance
                for (; open; open &= open - 1) {
                    const uint32_t v = (uint32_t)__ffs(open) - 1u;
                    if (d2_exact(spos[i], spos[a + v], g.L, g.half) < g.l2) links |= 1u << v;
                }
            }
            });
        }
        const uint64_t lm = __ballot(links != 0u);
        if (!lm) continue;
        // queue the links (any order)
        if (lane == 0) s_n[w] = queued;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        if (links) {
            uint32_t at = atomicAdd(&s_n[w], (uint32_t)__popc(links));
            for (uint32_t m = links; m; m &= m - 1) s_link[w][at++] = make_int2(i, (int)(a + (uint32_t)__ffs(m) - 1u));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        queued = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_n[w]);
        while (queued >= 64u) join(64u);
    }
    if (queued) join(queued);
}

constexpr int kRootsPer = 2;
// Roots of all members, read-only: nothing writes the forest in this pass, so
// every stored root is final (a compressing writer could otherwise replace a
// stored root with an older ancestor).
// The root of every particle's set into root[], and the smallest original
// index of every set into minorig[root] (one atomic per run of equal roots
// among consecutive lanes).  Two particles per thread, and only members' indices
// read: the time is the chain of loads (137 -> 101 us on the 256^3 box).
__global__ __launch_bounds__(kBlock) void k_fof_roots(int64_t n, const int32_t *__restrict__ parent,
                                                      const float4 *__restrict__ spos,
                                                      int32_t *__restrict__ root,
                                                      int32_t *__restrict__ minorig) {
    const int64_t i0 = (int64_t)blockIdx.x * (kRootsPer * kBlock) + threadIdx.x;
    int r[kRootsPer], p[kRootsPer];
    int32_t o[kRootsPer];
#pragma unroll
    for (int u = 0; u < kRootsPer; u++) r[u] = i0 + u * kBlock < n ? parent[i0 + u * kBlock] : -1;
#pragma unroll
    for (int u = 0; u < kRootsPer; u++) {
        o[u] = 0x7fffffff;
        p[u] = r[u];
        if (r[u] >= 0) {
            o[u] = (int32_t)orig_of(spos[i0 + u * kBlock]);
            p[u] = parent[r[u]];
        }
    }
#pragma unroll
    for (int u = 0; u < kRootsPer; u++) {
        while (p[u] != r[u]) {
            r[u] = p[u];
            p[u] = parent[r[u]];
        }
        if (i0 + u * kBlock < n) root[i0 + u * kBlock] = r[u];
        const WaveRun run = wave_run(r[u]);
        const int32_t m = wave_run_min(o[u], run);
        if (r[u] >= 0 && run.rank == 0) atomicMin(&minorig[r[u]], m);
    }
}

// One atomic per run of equal keys among consecutive lanes (every lane of the
// wavefront takes part; key < 0: none).
__device__ __forceinline__ void count_members(int key, uint32_t *__restrict__ gcnt) {
    const WaveRun r = wave_run(key);
    if (key >= 0 && r.rank == 0) atomicAdd(&gcnt[key], (uint32_t)r.len);
}

// Group key (smallest original index of the group, in the call's numbering)
// per sorted particle, the members of every key counted, and the L0 label
// (box-local) in original order.  A key outside [0, n) would be an internal
// error; it is flagged instead of being used as an index.
__global__ __launch_bounds__(kBlock) void k_fof_keys(int64_t n, Boxes bx, const int32_t *__restrict__ root,
                                                     const int32_t *__restrict__ minorig,
                                                     const float4 *__restrict__ spos,
                                                     int32_t *__restrict__ gkey,
                                                     uint32_t *__restrict__ gcnt,
                                                     int32_t *__restrict__ l0_out,
                                                     int32_t *__restrict__ err) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int k = -1;
    if (i < n) {
        const int r = root[i];
        k = r < 0 ? -1 : minorig[r];
        if (k >= n) {
            flag_error(err, 4, box_of(bx, (uint32_t)i));
            k = -1;
        }
        gkey[i] = k;
        if (l0_out)
            l0_out[orig_of(spos[i])] = k < 0 ? 0 : k + 1 - (int)bx.geo[box_of(bx, (uint32_t)i)].orig_base;
    }
    count_members(k, gcnt);
}

// Label and density of each particle side by side, in input order (one
// coalesced pass), so that the gather into sorted order below reads one
// 8-byte element per particle instead of two random 4-byte ones.  The member
// counts start here.
__global__ __launch_bounds__(kBlock) void k_pack_labels(int64_t n, const int32_t *__restrict__ l0_in,
                                                        const float *__restrict__ dens_in,
                                                        uint2 *__restrict__ packed,
                                                        uint32_t *__restrict__ gcnt,
                                                        uint64_t *clock) {
    stamp(clock);
    const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= n) return;
    packed[o] = make_uint2((uint32_t)l0_in[o], __float_as_uint(dens_in[o]));
    gcnt[o] = 0u;
}

// Group keys from caller-provided labels (1..n, 0 = none) and the caller's
// densities, in sorted order, and the members of every key counted.
__global__ __launch_bounds__(kBlock) void k_keys_from_labels(int64_t n, Boxes bx,
                                                             const uint2 *__restrict__ packed,
                                                             const float4 *__restrict__ spos,
                                                             int32_t *__restrict__ gkey,
                                                             float *__restrict__ dens_s,
                                                             uint32_t *__restrict__ gcnt,
                                                             int32_t *__restrict__ err) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int key = -1;
    if (i < n) {
        const int box = box_of(bx, (uint32_t)i);
        const Geo &g = bx.geo[box];
        const uint2 v = packed[orig_of(spos[i])];
        int32_t lab = (int32_t)v.x;
        // the candidate search orders densities by their bit patterns, which
        // matches their values for non-negative numbers only: -0 becomes +0
        // (the same value), NaN and negative values are rejected
        uint32_t db = v.y == 0x80000000u ? 0u : v.y;
        if ((db >> 31) != 0u || (db & 0x7fffffffu) > 0x7f800000u) {
            flag_error(err, 16, box);
            db = 0u;
        }
        dens_s[i] = __uint_as_float(db);
        // labels are box-local (1 .. box size, 0 = outside every group)
        if (lab < 0 || (int64_t)lab > g.n) {
            flag_error(err, 2, box);
            lab = 0;
        }
        key = lab > 0 ? lab - 1 + (int32_t)g.orig_base : -1;
        gkey[i] = key;
    }
    count_members(key, gcnt);
}

}  // namespace

void launch_fof(int64_t n, const Boxes &bx, Work &w, hipStream_t s) {
    const SegList sl = seg_list(n, w);
    // the first members of the dense sub-cells go to the sub-cell maxima's
    // argument table (free until the candidate stage)
    const int per = list_per(n);
    hipLaunchKernelGGL(per == 2 ? k_fof_phase_a<2> : k_fof_phase_a<1>, grid((n + per - 1) / per), dim3(kBlock), 0, s, n, bx, w.marks, w.ssub, w.subtab,
                       w.dens_s, w.parent, w.subarg, w.minorig, w.gcnt, sl, w.clock + kClockFof);
    if (w.ndcells > 0) {
        const dim3 cells((unsigned)((w.ndcells + kHalves - 1) / kHalves));
        hipLaunchKernelGGL(k_fof_cells, cells, dim3(kBlock), kHalves * bx.nsub_max * sizeof(float4), s, w.ndcells, bx,
                           w.sloc, w.subtab, w.subarg, w.parent);
        hipLaunchKernelGGL(k_fof_faces, cells, dim3(kBlock), 0, s, w.ndcells, bx, w.dcells, w.cells, w.sloc,
                           w.subtab, w.subarg, w.parent);
        hipLaunchKernelGGL(k_fof_cell_roots, cells, dim3(kBlock), 0, s, w.ndcells, bx, w.subtab,
                           w.subarg, w.parent);
    }
    if (w.nchunks > 0) {
        // one wavefront per workgroup: chunk costs differ widely, and a
        // finished wavefront's slot is free at once.  Three per chunk up to
        // three quarters of the wavefronts the chip holds: with 4209 chunks 66 us
        // became 44 and with 332 30 became 23, but with 9699 68 became 87.  (The
        // line is one box's: in 64 boxes, whose chains are longer, 9082 chunks
        // would still gain, 82 to 64 us, which the chunk count does not tell.)
        const int parts = w.nchunks <= 24 * (int64_t)(w.ncu > 0 ? w.ncu : 1) ? 3 : 1;
        hipLaunchKernelGGL(k_fof_dense, dim3((unsigned)(w.nchunks * parts)), dim3(64), 0, s, w.nchunks, xcd_tile(bx), parts, n, bx,
                           w.chunks, w.sloc, w.spos, w.cells, w.marks, w.subtab, w.subarg, w.dens_s, w.parent);
    }
    if (w.nsparse > 0)
        // one member in ten sparse particles: sixteen lanes per 8 particles at
        // most, and no more than fit the chip
        hipLaunchKernelGGL(k_fof_sparse, dim3(seg_blocks(sl, w.nsparse, 16, 8, 8 * (int64_t)(w.ncu > 0 ? w.ncu : 1))),
                           dim3(kBlock), 0, s, sl, bx, w.sloc, w.spos, w.cells, w.dens_s, w.parent);
    // roots go to the owner array (free until the assignment stage)
    hipLaunchKernelGGL(k_fof_roots, grid((n + kRootsPer - 1) / kRootsPer), dim3(kBlock), 0, s, n, w.parent, w.spos, w.owner, w.minorig);
}

void launch_fof_labels(int64_t n, const Boxes &bx, Work &w, int32_t *l0_out, hipStream_t s) {
    hipLaunchKernelGGL(k_fof_keys, grid(n), dim3(kBlock), 0, s, n, bx, w.owner, w.minorig, w.spos, w.gkey,
                       w.gcnt, l0_out, w.err);
}

void launch_keys_from_labels(const int32_t *l0_in, const float *dens_in, int64_t n, const Boxes &bx, Work &w,
                             hipStream_t s) {
    // the packed copy lives in the second radix key array (free after binning)
    uint2 *packed = reinterpret_cast<uint2 *>(w.rkey[1]);
    hipLaunchKernelGGL(k_pack_labels, grid(n), dim3(kBlock), 0, s, n, l0_in, dens_in, packed, w.gcnt,
                       w.clock + kClockDensity);
    hipLaunchKernelGGL(k_keys_from_labels, grid(n), dim3(kBlock), 0, s, n, bx, packed, w.spos, w.gkey, w.dens_s,
                       w.gcnt, w.err);
}

}  // namespace hf
