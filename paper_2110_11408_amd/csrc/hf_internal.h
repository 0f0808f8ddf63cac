// Internal declarations of libhf: the geometry/constant block passed to every
// kernel, device helpers for the canonical predicates, and the stage launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hf.h"

namespace hf {

constexpr int kBlock = 256;
constexpr int kDenseMin = 8;   // a cell with at least this many particles is "dense"
constexpr int kRadBins = 2048; // radial bins of the threshold-radius search by bins

// Constants of one periodic box, computed on the host (see hf_derived).
struct Geo {
    double L, half;        // periodic side and L/2 (minimum-image test)
    double cell, inv_cell; // binning cell side (>= max(b, l)) and its inverse
    double inv_b;          // 1/b: local coordinates are stored in units of b
    double inv_b2;         // 1/b^2: FP64 kernel weights 1 - r^2/b^2
    float cellb;           // cell / b in FP32 (image offset of a neighbour cell)
    int nc;                // cells per side (>= 3)
    double inv_nc;         // 1 / nc (cell coordinates from a cell id)
    int ksub;              // sub-cells per cell side (sub-cell diagonal < l)
    int nsub;              // ksub^3
    double inv_sub;        // ksub / cell
    int face_sub_in_b;     // any two points of face-adjacent sub-cells are closer than b
    double b2, l2;         // FP64 squared radii of the peak test and of FoF links
    float l2b_lo, l2b_hi;  // (l/b)^2 shrunk / grown by the FP32 prefilter margin
    float b2b_hi;          // 1 grown by the same margin (peak test, units of b^2)
    double norm;           // density normalisation 15/(8 pi b^3 nbar)
    int self_count;
    double dl0;            // L0 density threshold
    double floor_nuc;      // nucleation floor
    double K, K2, A6, C3;  // R^3 = i/K; alpha^6; c_Roche^3
    double rbin;           // radial bin width of the threshold-radius search by bins
    int n_l1_min;
    float particle_mass;
    // the box's place among the boxes of one call
    uint32_t cell_base;    // its first cell in the call's cell numbering
    uint32_t orig_base;    // its first particle (input and sorted order alike)
    int64_t n;             // its particles
    hf_halo *halos;        // its halo table (device), or null
    int64_t halo_cap;      // rows of that table
};

// The boxes of one call.  Particles and cells of all boxes are numbered
// together, box after box, so box b holds particles [base[b], base[b + 1])
// both in input order and after the sort (the sort key leads with the cell,
// and box b's cells follow box b - 1's), and cells
// [geo[b].cell_base, geo[b + 1].cell_base).  Labels are 1 + an index inside
// the box.
struct Boxes {
    const Geo *geo;        // device [nbox]
    const uint32_t *base;  // device [nbox + 1]: first particle of each box, then the total
    int nbox;
    int nsub_max;          // largest ksub^3: the sort-key stride of a cell and the row
                           // length - 1 of the dense-cell sub-tables
    const int32_t *btab;   // device (nbox > 1): btab[k] = box of particle k << bshift
    int bshift;
};

// Box of particle i (input or sorted order): the box of the table bucket that
// holds i, then forward over the box starts inside the bucket (a step or two:
// the table has several buckets per box on average).  No load when there is
// one box.
__device__ __forceinline__ int box_of(const Boxes &bx, uint32_t i) {
    if (bx.nbox <= 1) return 0;
    int b = bx.btab[i >> bx.bshift];
    while (b + 1 < bx.nbox && bx.base[b + 1] <= i) b++;
    return b;
}

// The constants of box b (the same in every lane) in registers: word by word
// through the constant address space, so scalar loads also where stores of the
// kernel could lie in between (nothing writes the tables while kernels run);
// words that are not used are not loaded.
__device__ __forceinline__ Geo box_constants(const Boxes &bx, int b) {
    typedef const __attribute__((address_space(4))) uint32_t *Words;
    const Words p = (Words)(uintptr_t)(bx.geo + b);
    static_assert(sizeof(Geo) % 4 == 0, "Geo is a run of words");
    uint32_t words[sizeof(Geo) / 4];
#pragma unroll
    for (size_t k = 0; k < sizeof(Geo) / 4; k++) words[k] = p[k];
    Geo g;
    __builtin_memcpy(&g, words, sizeof(Geo));
    return g;
}

// f(constants of box b) for every lane, one box of the wavefront at a time
// (nearly always one in all), with the box index in a scalar register, so that
// the constants come with scalar loads.  With an index per lane every constant
// is a vector load of its own, again in every loop that uses it.  The empty asm
// hides that the scalar index equals the lane's, which the compiler would put
// back in its place.
template <class F>
__device__ __forceinline__ void per_box(const Boxes &bx, int b, F f) {
    for (uint64_t todo = __ballot(true); todo;) {
        const int b1 = __builtin_amdgcn_readlane(b, (int)__builtin_ctzll(todo));
        int b0 = b1;
        asm volatile("" : "+s"(b0));
        const bool mine = b == b1;
        if (mine) f(box_constants(bx, b0));
        todo &= ~__ballot(mine);
    }
}

// ---------------------------------------------------------------- predicates
// Canonical minimum-image squared distance in FP64: the same sequence of IEEE
// operations as the definition (differences of the float32 inputs promoted to
// double, one image fold per axis, (xx + yy) + zz) with no fused multiply-add.
__device__ __forceinline__ double d2_exact(float4 a, float4 b, double L, double half) {
#pragma clang fp contract(off)
    double dx = (double)b.x - (double)a.x;
    double dy = (double)b.y - (double)a.y;
    double dz = (double)b.z - (double)a.z;
    if (dx > half) dx -= L; else if (dx < -half) dx += L;
    if (dy > half) dy -= L; else if (dy < -half) dy += L;
    if (dz > half) dz -= L; else if (dz < -half) dz += L;
    double xx = dx * dx;
    double yy = dy * dy;
    double zz = dz * dz;
    double s = xx + yy;
    return s + zz;
}

__device__ __forceinline__ double e3(double e) {
#pragma clang fp contract(off)
    double ee = e * e;
    return ee * e;
}

__device__ __forceinline__ double ii(int64_t k) {
#pragma clang fp contract(off)
    double x = (double)k;
    return x * x;
}

__device__ __forceinline__ uint32_t orig_of(float4 p) { return __float_as_uint(p.w); }

// "Denser" total order of nuclei: higher density, ties to the lower index.
__device__ __forceinline__ bool denser(float da, uint32_t ia, float db, uint32_t ib) {
    return da > db || (da == db && ia < ib);
}

// Workgroups are dispatched to the 8 XCDs round-robin (workgroup b runs on XCD
// b mod 8), and each XCD has its own L2.  Work lists are in spatial order, so a
// kernel whose neighbours overlap maps workgroup b to a logical index such that
// every XCD gets one contiguous slice of the list and its L2 sees the reuse.
constexpr unsigned kXcds = 8;

__device__ __forceinline__ unsigned xcd_block() {
    const unsigned b = blockIdx.x, nb = gridDim.x;
    const unsigned per = nb / kXcds, rem = nb % kXcds;
    const unsigned x = b % kXcds, k = b / kXcds;
    const unsigned start = x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per;
    return start + k;
}

// The same with slices of `tile` blocks dealt to the XCDs in turn, for lists whose
// parts differ in cost: one contiguous part per XCD leaves some XCDs with the
// chunks of the largest haloes.  The density kernels and the record buckets take
// slices of 16 (3.1M particles: k_density_dense 330 us contiguous, 297 in slices of
// 64, 282 of 4 or 16; 1.0M: k_density_rows 125, 117, 114; 512^3: 29.6, 28.2, 28.2
// ms; 256^3: 1.73, 1.73, 1.73), the FoF chunks slices of 64 and in a batch only (96
// boxes: k_fof_dense 3.42 -> 3.03 ms): in one box their links run along the slices,
// and contiguous ones are better (64^3: 44 us against 58; 512^3: 8.21 ms against
// 8.55).
constexpr unsigned kXcdTile = 16;
inline unsigned xcd_tile(const Boxes &bx) { return bx.nbox > 1 ? 64u : 0u; }
__device__ __forceinline__ unsigned xcd_tile_block(unsigned tile) {
    if (tile == 0u) return xcd_block();
    const unsigned b = blockIdx.x, whole = gridDim.x / (kXcds * tile) * (kXcds * tile);
    if (b >= whole) return b;
    const unsigned x = b % kXcds, k = b / kXcds;
    return (k / tile * kXcds + x) * tile + k % tile;
}

// FP32 squared distance for the prefilters (one multiply and two fused
// multiply-adds); their margins are far above the rounding of either form.
__device__ __forceinline__ float d2_f32(float dx, float dy, float dz) {
    return fmaf(dx, dx, fmaf(dy, dy, dz * dz));
}

// Value of lane L (L wave-uniform): a v_readlane into a scalar register,
// without the LDS round trip of a general shuffle.
__device__ __forceinline__ int lane_get(int v, int L) { return __builtin_amdgcn_readlane(v, L); }
__device__ __forceinline__ uint32_t lane_get(uint32_t v, int L) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, L);
}
__device__ __forceinline__ float lane_get(float v, int L) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), L));
}

// Scans and reductions over the 64 lanes (all active) in data-parallel-primitive
// moves: shifts by 1, 2, 4 and 8 lanes within the rows of 16, then the last lane
// of row 0 (2) to row 1 (3), and of the lower half to the upper one.  A lane
// without a source takes `none`.
template <int kCtrl, int kRows>
__device__ __forceinline__ int dpp_move(int none, int v) {
    return __builtin_amdgcn_update_dpp(none, v, kCtrl, kRows, 0xf, false);
}
template <typename Op>
__device__ __forceinline__ int dpp_scan(int v, Op op) {
    v = op(v, [](int none, int x) { return dpp_move<0x111, 0xf>(none, x); });
    v = op(v, [](int none, int x) { return dpp_move<0x112, 0xf>(none, x); });
    v = op(v, [](int none, int x) { return dpp_move<0x114, 0xf>(none, x); });
    v = op(v, [](int none, int x) { return dpp_move<0x118, 0xf>(none, x); });
    v = op(v, [](int none, int x) { return dpp_move<0x142, 0xa>(none, x); });
    return op(v, [](int none, int x) { return dpp_move<0x143, 0xc>(none, x); });
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    return (uint32_t)dpp_scan((int)v, [](int x, auto from) { return x + from(0, x); });
}
__device__ __forceinline__ float wave_min(float v) {
    const int m = dpp_scan(__float_as_int(v), [](int x, auto from) {
        return __float_as_int(fminf(__int_as_float(x), __int_as_float(from(x, x))));
    });
    return lane_get(__int_as_float(m), 63);
}
__device__ __forceinline__ float wave_max(float v) {
    const int m = dpp_scan(__float_as_int(v), [](int x, auto from) {
        return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(from(x, x))));
    });
    return lane_get(__int_as_float(m), 63);
}

// a / d for 0 <= a < 2^16 and 1 <= d <= 256 from FP32, given inv_d = 1/d:
// (a + 1/2) / d is at least 1/(2d) away from every integer and its FP32
// product with inv_d is within a few ulps of it, far less, so the truncation
// is the integer quotient (a few instructions instead of an integer division
// by a variable; checked exhaustively over that range).
__device__ __forceinline__ int div_small(int a, float inv_d) { return (int)(((float)a + 0.5f) * inv_d); }

__device__ __forceinline__ int wrapc(int c, int nc) {
    return c < 0 ? c + nc : (c >= nc ? c - nc : c);
}

// x / nc for a cell id x < 2^32: the FP64 product with 1/nc is within far
// less than one of x / nc (x is exact in FP64), so its truncation is the
// quotient or one below it; one comparison corrects that (and, for safety, one
// above).
__device__ __forceinline__ uint32_t div_nc(uint32_t x, const Geo &g) {
    uint32_t q = (uint32_t)((double)x * g.inv_nc);
    const uint64_t nc = (uint64_t)g.nc;
    if ((uint64_t)(q + 1) * nc <= (uint64_t)x) q++;
    else if ((uint64_t)q * nc > (uint64_t)x) q--;
    return q;
}

// Coordinates inside its box of cell c (the call's numbering) of box g.
__device__ __forceinline__ void cell_xyz(const Geo &g, uint32_t c, int &cx, int &cy, int &cz) {
    const uint32_t lc = c - g.cell_base, nc = (uint32_t)g.nc;
    const uint32_t q = div_nc(lc, g), q2 = div_nc(q, g);
    cx = (int)(lc - q * nc);
    cy = (int)(q - q2 * nc);
    cz = (int)q2;
}

// The cell at coordinates (x, y, z) of box g, each wrapped once (one cell
// beyond a face at most), in the call's numbering.
__device__ __forceinline__ uint32_t cell_id(const Geo &g, int x, int y, int z) {
    const int nc = g.nc;
    return g.cell_base + ((uint32_t)wrapc(z, nc) * (uint32_t)nc + (uint32_t)wrapc(y, nc)) * (uint32_t)nc +
           (uint32_t)wrapc(x, nc);
}

// Record error bit `bit` for box `box` (err[0] collects the bits, err[1] the
// smallest box that raised one).
__device__ __forceinline__ void flag_error(int32_t *err, int32_t bit, int box) {
    atomicOr(err, bit);
    atomicMin(err + 1, box);
}

__device__ __forceinline__ bool is_member(const float *dens_s, int64_t j, double dl0) {
    return (double)dens_s[j] > dl0;
}

// Runs of equal keys among consecutive lanes of a wavefront: the lane of the
// run's first element, this lane's rank in the run, and the run length.  Used
// to aggregate atomics on sorted data (one atomic per run instead of per lane).
struct WaveRun {
    int head, rank, len;
};

__device__ __forceinline__ WaveRun wave_run(int key) {
    const int lane = threadIdx.x & 63;
    const int prev = __shfl_up(key, 1, 64);
    const bool is_head = lane == 0 || prev != key;
    const uint64_t heads = __ballot(is_head);
    const uint64_t le = lane == 63 ? ~0ull : ((1ull << (lane + 1)) - 1ull);
    const int head = 63 - __clzll(heads & le);
    const uint64_t upto_head = head == 63 ? ~0ull : ((2ull << head) - 1ull);
    const uint64_t above = heads & ~upto_head;
    const int next = above ? __ffsll((unsigned long long)above) - 1 : 64;
    return WaveRun{head, lane - head, next - head};
}

// Minimum of v over the lane's run (valid in the run's head lane).
__device__ __forceinline__ int32_t wave_run_min(int32_t v, const WaveRun &r) {
    const int lane = threadIdx.x & 63;
    const int end = r.head + r.len;
    for (int d = 1; d < 64; d <<= 1) {
        int32_t o = __shfl_down(v, d, 64);
        if (lane + d < end) v = min(v, o);
    }
    return v;
}

// --------------------------------------------------------------- workspace
// Bits of the sorted particles, 64 to a word: head of a dense chunk, head of a
// dense cell, in a sparse cell, head of a cell; and the sparse particles and the
// dense cells before each word.
struct Marks {
    uint64_t *chunk, *dcell, *sparse, *head;
    uint32_t *before, *dbefore;
};
__device__ __forceinline__ bool is_sparse(const Marks &m, int64_t i) { return (m.sparse[i >> 6] >> (i & 63)) & 1ull; }
// Number of the dense cell that holds particle i (of a dense cell).
__device__ __forceinline__ uint32_t dense_ordinal(const Marks &m, uint32_t i) {
    return m.dbefore[i >> 6] + (uint32_t)__popcll(m.dcell[i >> 6] & (~0ull >> (63u - (i & 63u)))) - 1u;
}
// End of the chunk of at most 64 particles that starts at h: the next cell's
// head, which lies in h's word or the next one if it is among the 64.
__device__ __forceinline__ uint32_t chunk_end(const Marks &m, uint32_t h, int64_t n) {
    const uint32_t w = h >> 6;
    const bool more = (int64_t)(w + 1u) * 64 < n;
    const uint64_t m0 = m.head[w] & ~(~0ull >> (63u - (h & 63u))), m1 = more ? m.head[w + 1u] : 0ull;
    const uint32_t last = (uint32_t)min((int64_t)h + 64, n);
    if (m0) return min(last, w * 64u + (uint32_t)__builtin_ctzll(m0));
    if (m1) return min(last, (w + 1u) * 64u + (uint32_t)__builtin_ctzll(m1));
    return last;
}
// Place of sparse particle i in the sparse list.
__device__ __forceinline__ uint32_t sparse_ordinal(const Marks &m, uint32_t i) {
    return m.before[i >> 6] + (uint32_t)__popcll(m.sparse[i >> 6] & ((1ull << (i & 63u)) - 1ull));
}

// The grid as an index of the cells that hold particles, which are numbered in
// order: a word per 32 cells with a bit for each such cell and the number of the
// word's first one (0 in a word without one), and per number the first particle
// (start, with the end after the last) and, for dense cells, the number among
// those.  A first-particle entry per cell is one load less to look a cell up, but
// nearly all cells are empty on a cosmological box: 2 GB with the dense cells'
// map on the 256^3 box, written in 280 us and missed by every gather, against
// 62 MB of words.  The density kernel of the sparse cells read 2.0 GB with it and
// reads 0.66 GB now; a find on that box went from 7456 to 7211 us, the density of
// 3.1M particles from 844 to 739 us.
struct Cells {
    uint2 *occ;
    uint32_t *start, *dmap;
};
constexpr int kOccCells = 32;  // cells per word
inline int64_t occ_words(int64_t ncell) { return ncell / kOccCells + 1; }
// Cell c's word gives the number of cell c, or of the next cell of the word that
// holds particles; `has`: whether c does.
__device__ __forceinline__ uint32_t cell_number(const uint2 &word, uint32_t c, uint32_t &has) {
    const uint32_t b = c & (uint32_t)(kOccCells - 1);
    has = (word.x >> b) & 1u;
    return word.y + (uint32_t)__popc(word.x & ((1u << b) - 1u));
}
// Words in a row, loaded at once (4-byte aligned).
struct alignas(4) Words4 {
    uint32_t v[4];
};
// The particles [a, e) of cell c (a = e when it is empty); returns its number.
__device__ __forceinline__ uint32_t cell_range(const Cells &cells, const uint2 &word, uint32_t c, uint32_t &a,
                                               uint32_t &e) {
    uint32_t has;
    const uint32_t o = cell_number(word, c, has);
    a = e = 0u;
    if (has) {
        a = cells.start[o];
        e = cells.start[o + 1u];
    }
    return o;
}
__device__ __forceinline__ uint32_t cell_range(const Cells &cells, uint32_t c, uint32_t &a, uint32_t &e) {
    return cell_range(cells, cells.occ[c / kOccCells], c, a, e);
}

// Entries of a table of the dense cells' sub-cells (at most n / kDenseMin dense
// cells, a row of nsub + 1 entries each).
inline int64_t sub_entries(int64_t n, int nsub) { return (n / kDenseMin + 1) * (nsub + 1); }

struct Work {
    // binning
    Cells cells;                     // cell -> particles, dense-cell number
    uint64_t *rkey[2];               // radix sort keys (ping-pong, rkey[1] = rkey[0] + n); reused after binning
    uint32_t *rval[2];               // radix sort payload: original index
    uint32_t *rhist, *rscan;         // per-pass [digit][tile] counts and their scan
    uint16_t *ssub;
    float4 *spos, *sloc;
    float4 *pq;                      // density only: cell-centred (x, y, z, -|x|^2), n + 32 entries
    // work decomposition (dense chunks, dense cells, sparse particles)
    uint32_t *scell;                 // cell of every sorted particle
    Marks marks;                     // dense chunk and cell heads, sparse particles, cell heads
    uint32_t *tmp_a, *tmp_b, *tmp_c, *tmp_d;  // scratch of n + 1 words each, in one run
    int32_t *chunks, *sparse;
    uint32_t *dcells;
    float4 *rec2;                                      // sub_entries records, over the three tables:
    uint32_t *subtab;                                  // first particle per dense sub-cell
    uint64_t *submax;                                  // densest particle per dense sub-cell
    int32_t *subarg;
    int32_t *hardlist;                                 // candidate tests left after stage 1
    int64_t nchunks, ndcells, nsparse, nhard, nlate;
    int ncu;                         // compute units (grids of the persistent kernels)
    bool radius_bins;                // R_L1 by radial bins instead of the whole-group histogram
    // density / FoF / groups (sorted order unless noted)
    float *dens_s;
    int32_t *parent, *minorig, *gkey, *gid_of, *owner;
    uint32_t *gcnt, *goff, *gidx;                     // key space [0, n]
    int32_t *mem;                                     // members grouped by group
    int32_t *g_start, *g_size, *g_label;              // per group
    uint32_t *gccnt, *gcoff, *gcfill;                  // candidates per group
    int32_t *glist;                                    // groups with candidates
    int32_t *cand, *cand_sorted;                       // candidates
    int32_t *h_nuc, *h_ienc, *h_gid, *g_nh;            // halo slots (= candidate slots)
    uint32_t *h_count;
    uint32_t *tflag, *tpos;                            // table rows: a bit per original index, and the
                                                       // prefix sum of the words' set bits
    uint32_t *scan_tmp;
    double *gcom;                    // halo statistics only: centres per group (6 doubles)
    int32_t *ordk;                   // halo statistics only: group ordinal per key
    int32_t *counters;                                 // small device counters
    int32_t *err;                    // [0] error bits, [1] smallest box with an error
    Geo *geo, *geo2;                 // the boxes' constants (geo2: level 2, halo statistics only)
    uint32_t *base;                  // first particle of every box, then the total
    int32_t *btab;                   // box of every 2^bshift-th particle (Boxes::btab)
    uint32_t *host;                                    // the lane's pinned host words (read_words)
    uint64_t *clock;                 // pinned: the device's wall clock at the stages' starts (kClock*)
};

// Stage times: the first kernel of a stage writes the device's wall clock to
// the stage's pinned word, and the host reads the words after the wait that ends
// the call.  (An event at every stage is a packet between two kernels and a host
// call each, and its elapsed time another; with them, two table copies, three
// fills and a copy of the row counts a find of 20 000 particles took 417 us and
// one of 64^3 690 us, without 377 and 648.)  A stage that launches nothing leaves
// its word 0 and starts with the next one.
enum { kClockBin = 0, kClockDensity, kClockFof, kClockSegment, kClockCand, kClockAccept, kClockAssign,
       kClockOutput, kClockEnd, kClocks };
__device__ __forceinline__ void stamp(uint64_t *at) {
    if (at && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(at, (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A list that one kernel fills for the next, in nseg segments of `cap` entries:
// workgroup b appends to segment b mod nseg with one atomic, so no address
// sees more than a 64th of the workgroups (a flag per particle, a scan and a
// list kernel took 60 us on the 256^3 box, a count read back by the host
// another 25 us of an idle device).  Counters lie kSegStride words apart.
constexpr uint32_t kSegs = 64, kSegStride = 16;
struct SegList {
    int32_t *list;
    uint32_t *count;
    uint32_t nseg, cap;
};

// Appends i of the lanes with `take` (every thread of the kBlock takes part).
// (K particles per thread: the workgroup waits once for its atomic.)
template <int K>
__device__ __forceinline__ void seg_append(const SegList &sl, const bool (&take)[K], const int32_t (&i)[K]) {
    __shared__ uint32_t s_cnt[kBlock / 64], s_base;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t m[K];
    uint32_t mine = 0;
#pragma unroll
    for (int u = 0; u < K; u++) {
        m[u] = __ballot(take[u]);
        mine += (uint32_t)__popcll(m[u]);
    }
    if (lane == 0) s_cnt[w] = mine;
    __syncthreads();
    const uint32_t seg = blockIdx.x % sl.nseg;
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int x = 0; x < kBlock / 64; x++) t += s_cnt[x];
        s_base = t ? atomicAdd(sl.count + seg * kSegStride, t) : 0u;
    }
    __syncthreads();
    uint32_t at = s_base;
    for (int x = 0; x < w; x++) at += s_cnt[x];
#pragma unroll
    for (int u = 0; u < K; u++) {
        if (take[u]) sl.list[(int64_t)seg * sl.cap + at + (uint32_t)__popcll(m[u] & ((1ull << lane) - 1ull))] = i[u];
        at += (uint32_t)__popcll(m[u]);
    }
}

// The share of one of kBlock / W lane groups per workgroup in a list: entries
// k, k + step, ... of segment seg (none when k >= n).  The groups of a
// workgroup take consecutive entries of one segment: particles near each other,
// whose neighbourhoods overlap.  With all kSegs segments the grid is a multiple
// of kSegs workgroups and a workgroup serves a segment that the workgroups of
// its own XCD filled.
struct SegShare {
    uint32_t seg, k, step, n;
};
template <int W>
__device__ __forceinline__ SegShare seg_share(const SegList &sl) {
    constexpr uint32_t kGroups = kBlock / W;
    const uint32_t q = threadIdx.x / W;
    SegShare s;
    s.seg = blockIdx.x % sl.nseg;
    s.k = blockIdx.x / sl.nseg * kGroups + q;
    s.step = gridDim.x / sl.nseg * kGroups;
    s.n = sl.count[s.seg * kSegStride];
    return s;
}

// Words of Work::counters that several stages use (zero when a call begins).
enum {
    kCntChunks = 0,     // dense chunks
    kCntDcells = 1,     // dense cells
    kCntSparse = 3,     // particles of sparse cells
    kCntMidRest = 4,    // candidates of medium and of large groups to evaluate:
    kCntBigRest = 5,    // the groups' densest, and the others
    kCntLate = 6,       // the others of groups above accept_late members,
    kCntLateListed = 7, // and those of them listed
    kCntMidFirst = 9,
    kCntBigFirst = 11,
    kCntHard = 8,       // hard cases of the candidate stage
    kCntListed = 10,    // groups with candidates in glist
    kCntCand = 13,      // candidates
    kCntMembers = 14,   // members of all groups
    kCntGroups = 15     // groups
};

// Runs of words that the segmentation zeroes on its way for the stage after it.
struct SegClear {
    static constexpr int kRuns = 2;
    uint32_t *p[kRuns];
    int len[kRuns];
};

// Particles per thread of the kernels that fill a segmented list: two on large
// inputs, where twice the loads in flight hide their latency (k_cand_quick 191
// -> 152 us on the 256^3 box, k_fof_phase_a 167 -> 148), one where a wavefront's
// own chain is the time (20 000 particles: 4.7 us against 8.0; 2.6e5: 7.0 against
// 8.6; equal at 1.3e6).
inline int list_per(int64_t n) { return n > ((int64_t)1 << 20) ? 2 : 1; }

// The segmented list over n particles.  Its entries lie in the scratch arrays
// (4 n words in one run; the segments hold at most 2 (n + 255) words, and a
// single segment at most n), its counts in the radix counts (at least n / 8
// words, of which n / 16 + 16 are used).
inline SegList seg_list(int64_t n, const Work &w) {
    const int per_thread = list_per(n);
    const unsigned nb = (unsigned)((n + kBlock * per_thread - 1) / (kBlock * per_thread));
    SegList sl;
    sl.list = reinterpret_cast<int32_t *>(w.tmp_a);
    sl.count = w.rhist;
    sl.nseg = nb < kSegs ? nb : kSegs;
    sl.cap = (nb + sl.nseg - 1) / sl.nseg * (unsigned)(kBlock * per_thread);
    return sl;
}
// Workgroups whose lane groups of W share a segmented list of n particles'
// entries: about `most` of them, no more than one group per `per` particles, and
// a multiple of the segment count (at least one workgroup per segment).
inline unsigned seg_blocks(const SegList &sl, int64_t n, int W, int64_t per, int64_t most) {
    const int groups = kBlock / W;
    int64_t b = (n / per + groups - 1) / groups;
    if (b > most) b = most;
    const int64_t each = b / sl.nseg;
    return (unsigned)(sl.nseg * (each > 0 ? each : 1));
}

// ------------------------------------------------------------------ launchers
// Device words to read back to the host in one go.
struct WordSrc {
    static constexpr int kMax = 8;
    const uint32_t *p[kMax];
};
// One small kernel copies *src.p[0..k) into the pinned host buffer `host`
// (at least kMax words), the stream is synchronized and out[0..k) receives
// the values: one dispatch and one wait for all the counts a step needs.
hipError_t read_words(const WordSrc &src, int k, uint32_t *host, uint32_t *out, hipStream_t s,
                      uint64_t *clock = nullptr);
// Up to four word arrays copied from pinned host memory to the device, the
// call's counters and error words cleared and its first stamp taken, in one
// launch.
struct BeginCopy {
    const uint32_t *src;  // pinned: the arrays one after the other
    uint32_t *dst[4];
    uint32_t words[4];
};
hipError_t begin_call(const BeginCopy &c, int32_t *counters, int32_t *err, uint64_t *clock, hipStream_t s);
// The same in two halves: the copy is enqueued on s, and the words are read
// once the caller has waited for it (an event recorded right after it), so
// that later work can be enqueued first.
// (clock: a stage stamp to take as well, or null.)
hipError_t publish_words(const WordSrc &src, int k, uint32_t *host, hipStream_t s, uint64_t *clock = nullptr);
void collect_words(const uint32_t *host, int k, uint32_t *out);
void fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s);
void fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s);
// Exclusive scan: out[0..n] with out[n] = total.  tmp: a word per 4096 elements.
void scan_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp, hipStream_t s);
// Exclusive scan of the number of set bits of every word (same layout and tmp).
void scan_bits_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp, hipStream_t s);
// Words of Work::scan_tmp for n particles.
int64_t scan_tmp_words(int64_t n);

// Every launcher works on all boxes of the call at once: n is the particle
// total, bx the boxes (device tables), ncell the cell total.
void launch_bin(const float *pos, int64_t n, int64_t ncell, const Boxes &bx, Work &w, hipStream_t s);
// Level 2 summaries and position statistics after an L2 pass (stats.hip; one
// box, g its constants).
void launch_halo_stats(int64_t n, int64_t G, int64_t M, const Geo &g, double particle_mass, const float *pos,
                       const int32_t *halo_id, Work &w, hf_halo_summary *out, int32_t *group_start,
                       int32_t *group_members, hipStream_t s);
// Length of the radix count arrays for n particles.
int64_t radix_hist_len(int64_t n);
// Tiles of the kernels that mark and list n sorted particles.
int64_t bin_tiles(int64_t n);
// Stable LSD radix sort of n 64-bit keys a[] by their bits [lo, lo + bits),
// using b[] as the second buffer and w's count arrays; returns the buffer
// (a or b) that holds the result.
uint64_t *radix_sort_keys(uint64_t *a, uint64_t *b, int64_t n, int lo, int bits, Work &w, hipStream_t s);
void launch_subtab(int64_t n, const uint32_t *ndc_p, const Boxes &bx, Work &w, hipStream_t s);
void launch_density(int64_t n, const Boxes &bx, Work &w, float *dens_out, hipStream_t s);
void launch_count_pairs(int64_t n, const Boxes &bx, Work &w, unsigned long long *total, hipStream_t s);
void launch_gather_density(const float *dens_in, int64_t n, Work &w, hipStream_t s);
void launch_fof(int64_t n, const Boxes &bx, Work &w, hipStream_t s);
void launch_fof_labels(int64_t n, const Boxes &bx, Work &w, int32_t *l0_out, hipStream_t s);
void launch_keys_from_labels(const int32_t *l0_in, const float *dens_in, int64_t n, const Boxes &bx, Work &w,
                             hipStream_t s);
// From the keys and the member counts per key: the members by group and the
// group table; member and group counts go to w.counters.
void launch_segment(int64_t n, Work &w, hipStream_t s);
// Only the member and group counts.
void launch_segment_totals(int64_t n, Work &w, hipStream_t s);
SegClear candidates_clear(int64_t n, const Work &w);  // candidates.hip
// Extent check of the L0 groups (sets err bit 8 when a group spans half its
// box or more along an axis).
void launch_extent(int64_t n, const Boxes &bx, Work &w, hipStream_t s);
// Candidates (counts per group, first slot of every group, total in
// w.counters), then their slots in descending density per group and the groups
// with candidates in descending size (the largest first, over all boxes).
void launch_candidates(int64_t n, const Boxes &bx, Work &w, hipStream_t s);
void launch_candidate_lists(int64_t n, Work &w, hipStream_t s);
// Members from which on a group's other candidates wait for the densest one's
// enclosed count (k_accept_eval).
int accept_late(const Work &w);
// Groups with candidates (their count is read on the device; grid bound
// min(G, NC)); M = members of all groups, n = particles.
void launch_accept(int64_t n, int64_t G, int64_t NC, int64_t M, const Boxes &bx, Work &w, hipStream_t s);
void launch_assign(int64_t n, const Boxes &bx, Work &w, hipStream_t s);
void launch_output_flags(int64_t n, int64_t NC, const Boxes &bx, Work &w, hipStream_t s);
// halo_id / l0_out: device [n], box-local labels; dens_out: device [n], the
// densities (l0_out and dens_out may be null).  Each box's table goes to its
// Geo::halos when its rows fit in Geo::halo_cap.
void launch_output(int64_t n, int64_t NC, const Boxes &bx, Work &w, int32_t *halo_id, int32_t *l0_out,
                   float *dens_out, hipStream_t s);
// Ends a pass: every box's row count to `rows` (pinned host, [nbox]), the words
// of src to the lane's pinned words and the last stamp, in one launch.
void launch_finish(const Boxes &bx, const WordSrc &src, int k, Work &w, int64_t *rows, hipStream_t s);
// One box after launch_output: its n particles by table row of their halo
// (nrows rows, then the particles of no halo), ascending index within a row,
// into members [n]; halo_start [nrows + 1] receives each row's first position.
void launch_group_order(int64_t n, int64_t nrows, const int32_t *halo_id, Work &w, int32_t *members,
                        int64_t *halo_start, hipStream_t s);

}  // namespace hf
