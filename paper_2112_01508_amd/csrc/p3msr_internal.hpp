// Internal definitions shared by the HIP translation units of libp3msr.
//
// Data layout in HBM (all built per call from the caller's arrays):
//   sp[p]        double4 (x, y, z, w) of the p-th particle in tile -> subtile
//                order, positions wrapped into [0, box); w = mu (FP64 path) or
//                the bits of float mu in the low word (FP32 path)
//   perm[p]      original index of sorted particle p
//   sel[p]       receiver selector of sorted particle p (active flag or rung)
//   cell_start[c] first sorted index of fine cell c (c = tile*ns^3 + subtile),
//                cell_start[ncells] = n
//   rp[], rperm[] receivers (record, original index), subset-major, tile order
//   clusters[]   receiver groups of <= csize (8..64) particles inside one tile
//   items[]      (cluster, neighbour-tile range, subtile range) work units,
//                the items of one cluster consecutive
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

#include <cstddef>
#include <cstdint>

namespace p3m {

constexpr int kWave = 64;
constexpr int kScanBlock = 256;             // threads per scan block
constexpr int kScanPerThread = 16;          // elements per scan thread
constexpr int kScanTile = kScanBlock * kScanPerThread;
constexpr int kForceBlock = 256;            // 4 waves, each with its own work item
constexpr int kSupplierPad = 128;           // zeroed records after the sorted particles
constexpr int kFineSide = 8;                // fine order: 8x8x8 sub-cells per subtile
constexpr int kFineBins = kFineSide * kFineSide * kFineSide;
constexpr int kFineMin = 8;                 // subtiles with at most this many keep their order
constexpr int kFineBig = 1024;              // larger subtiles are ordered by a whole block
constexpr int kFineWaves = kFineBins / kWave;   // tiles (one per wave) per fine-order block
constexpr int kFinishWaves = 4;             // waves per block of the cluster box kernel
constexpr int kFinishLanes = 8;             // lanes per cluster in the box kernel
constexpr int kListCap = 224;               // screened supplier records per wave (LDS)
constexpr int kListCapF32 = 176;            // the same for the six-wave FP32 forward kernel
constexpr int kListCapAdjoint = 128;        // the same for the adjoint (entries carry weights)
constexpr int kListSlack = 32;              // records past the cap for look-ahead reads (3*8 used)

// Geometry of one call.  Tiles are cubes of side box/nt >= r_cut; each tile
// holds ns^3 subtiles; fine cells are the subtiles, nc = nt*ns per dimension.
struct Geom {
    double box, inv_box;
    double rc2;        // r_cut^2: the pair test is r^2 < rc2 (strict)
    double tile;       // tile side
    double sub;        // subtile side
    double inv_cell;   // nc / box
    double cull2;      // (r_cut + margin)^2 for conservative subtile culling
    double k1;         // 1 / (2 x_s)
    double k2;         // -log2(e) / (4 x_s^2): exp(-u^2) = 2^(r^2 k2)
    double kb;         // 1 / (2 sqrt(pi) x_s^3), Gaussian term of the pair Jacobian
    double x_s;
    int nt, ns, nc, ns3, nt3;
    float k1f, kbf;    // FP32 copies of k1 and kb
    float c2f;         // 1 / (4 x_s^2): t = u^2 = r^2 c2
    float c3f;         // 1 / (8 x_s^3): g(u) / r^3 = r^-3 + H(t) c3
    double c2, c3;     // FP64 copies of c2f and c3f
    double h64[18];    // FP64 H coefficients (kernel argument, so they sit in SGPRs)
    double eps_b;      // B-spline softening length (0: point particles)
    double eps_b2;     // eps_b^2: pairs with r^2 < eps_b2 take the softened form
    double inv_eps_b;  // 1 / eps_b
    double ks3, ks5;   // 32 / eps_b^3, 32 / eps_b^5
    float inv_eps_bf;  // FP32 copy of inv_eps_b
};

struct Cluster {
    int tile;     // tile index (tx*nt + ty)*nt + tz
    int subset;   // receiver subset (batched calls)
    int begin;    // first entry in rp / rperm
    int count;    // 1..csize receivers
    double lo[3]; // bounding box of the receivers (wrapped positions)
    double hi[3];
};

// Work item: receivers of one cluster against suppliers in neighbour tiles
// [t0, t1) of the 27-tile stencil (t = (ox+1)*9 + (oy+1)*3 + (oz+1)) and,
// when t1 == t0 + 1, only subtiles [s0, s1) of that tile.
struct Item {
    int cluster;
    int tiles;    // t0 | t1 << 8
    int subs;     // s0 | s1 << 16; kItemPart: part | parts << 16
    int sole;     // kItemSole: the only item of its cluster (its sums are stored, not
                  // added); kItemFirst: the cluster's first item; kItemPart: one of
                  // `parts` equal runs of the records of one tile of one subtile
};
constexpr int kItemSole = 1;
constexpr int kItemFirst = 2;
constexpr int kItemPart = 4;

struct Counters {
    unsigned long long interactions;
    unsigned long long candidates;
    unsigned long long steps;        // wave steps over suppliers
    unsigned long long screened;     // supplier records tested against cluster boxes
    unsigned long long rare;         // mutual kernel: wave steps that took the FP64 path
    unsigned long long scan_stall;   // single-pass scans whose look-back hit its poll limit
    unsigned long long pad[2];
};
static_assert(256 % sizeof(Counters) == 0, "Counters copies are 256 B apart");

// The pair kernels add their waves' counts into one Counters copy per XCD,
// each in a 256 B line of its own (the readers sum the copies): one copy for
// every wave would queue their atomics on one cache line at the end of the
// launch.
constexpr int kCounterCopies = 8;
constexpr int kCounterStride = 256 / sizeof(Counters);

enum SelKind { SEL_ALL = 0, SEL_MASK = 1, SEL_RUNG = 2 };

// ---- work items ---------------------------------------------------------------

// Greedy grouping of the 27 neighbour tiles into items of about `target`
// supplier candidates (before subtile culling); a tile holding more than
// `target` particles is split by subtile ranges, or, where a tile is one
// subtile and `split` is not 0, into runs of about `split` of its records.
// Without a split, at most 2 items per stencil tile plus one with one subtile
// per tile (a flush and the tile itself), at most 1 + ns^3 per tile plus one
// otherwise (plan_items_bound).  Splits add less than w / split items per
// cluster and tile of w particles, and a tile is in the stencils of at most
// 27 tiles, whose clusters number at most 27 + n / csize (split_items_bound).
// They are for small sets (kSplitMax): a halo that holds a good part of one
// has too few clusters to fill the GPU, and one of its items would walk the
// whole halo (120000 particles, half of them in one tile, FP32: 8.9 ms per
// call without, 2.8 ms with); in larger sets other clusters fill the GPU.
// A run is at least a kSplitRuns'th of the set (split_run), so the bound on
// the items grows with the set and not with its square, which took 1 GB near
// 2^20 particles or switched the split off (a million, 5 % of them in one tile,
// FP64: 6.7 ms, now 3.5 ms).  With 128 runs a set of 400000 of that shape takes
// 0.99 ms against 0.84 ms; without the limit, runs of `target`, 0.82 ms.
//
// HALF (pairs evaluated once, for both partners): only the upper half of the
// stencil, t = 13 .. 26, whose periodic mirror images are the lower half; in
// the own tile (t = 13) only the particles after the cluster count, and every
// cluster gets at least one item, so that its own pairs are evaluated.  The
// first item of a cluster carries kItemFirst.
// Upper bound on the items one cluster gets.
inline long long plan_items_bound(int ns3, int half) {
    const long long tiles = half ? 14 : 27;
    return tiles * (ns3 == 1 ? 2 : 1 + ns3) + 2;
}

constexpr int kSplitMax = 1 << 20;   // particles
constexpr int kSplitRuns = 256;
inline int split_run(long long n, int target) {
    const long long least = (n + kSplitRuns - 1) / kSplitRuns;
    return target > least ? target : (int)least;
}
inline long long split_items_bound(long long n, int csize, int run) {
    return (n / run) * (27 + n / csize);
}

// Particles of each stencil tile of the cluster [begin, begin + count) of
// `tile` that the plan counts.  All loads are issued before any is used: the
// plan is bound by their latency.
template <bool HALF>
__device__ __forceinline__ void plan_weights(int tile, int end, const int *__restrict__ cs,
                                             const Geom &g, int (&w)[27]) {
    constexpr int T0 = HALF ? 13 : 0;
    const int tx = tile / (g.nt * g.nt), ty = (tile / g.nt) % g.nt, tz = tile % g.nt;
    int lo[27], hi[27];
#pragma unroll
    for (int t = T0; t < 27; ++t) {
        int nx = tx + t / 9 - 1, ny = ty + (t / 3) % 3 - 1, nz = tz + t % 3 - 1;
        nx += nx < 0 ? g.nt : (nx >= g.nt ? -g.nt : 0);
        ny += ny < 0 ? g.nt : (ny >= g.nt ? -g.nt : 0);
        nz += nz < 0 ? g.nt : (nz >= g.nt ? -g.nt : 0);
        const size_t c = (size_t)((nx * g.nt + ny) * g.nt + nz) * g.ns3;
        lo[t] = cs[c];
        hi[t] = cs[c + g.ns3];
    }
    if constexpr (HALF) lo[13] = end;
#pragma unroll
    for (int t = T0; t < 27; ++t) w[t] = hi[t] - lo[t];
}

// The items of one cluster in order, each handed to emit(k, t0, t1, s0, s1,
// kItemPart or 0); returns their number.
template <bool HALF, class Emit>
__device__ __forceinline__ int plan_items(const int (&w)[27], int target, int ns3, int split,
                                          Emit emit) {
    constexpr int T0 = HALF ? 13 : 0;
    int n = 0, acc = 0, t0 = T0;
#pragma unroll
    for (int t = T0; t < 27; ++t) {
        if (w[t] > target) {
            if (acc > 0) emit(n++, t0, t, 0, ns3, 0);
            if (split) {
                const int parts = max(w[t] / split, 1);
                for (int q = 0; q < parts; ++q) emit(n++, t, t + 1, q, parts, kItemPart);
            } else {
                const int parts = min((w[t] + target - 1) / target, ns3);
                for (int q = 0; q < parts; ++q)
                    emit(n++, t, t + 1, q * ns3 / parts, (q + 1) * ns3 / parts, 0);
            }
            t0 = t + 1;
            acc = 0;
        } else if (acc + w[t] > target) {
            emit(n++, t0, t, 0, ns3, 0);
            t0 = t;
            acc = w[t];
        } else {
            if (acc == 0 && w[t] == 0) t0 = t + 1;   // skip leading empty tiles
            acc += w[t];
        }
    }
    if (acc > 0) emit(n++, t0, 27, 0, ns3, 0);
    if (HALF && n == 0) emit(n++, 13, 14, 0, ns3, 0);
    return n;
}

// ---- cell counting -----------------------------------------------------------

// Key and rank inside its cell of PPT consecutive-block particles per thread,
// with one global atomic per distinct cell of a block of kKeysThreads x PPT
// particles: the block's keys are counted in an LDS hash table first (a dense
// halo cell's particles, which share blocks, would otherwise hit one counter
// from every wave that holds any of them, and those atomics serialise on its
// address).  The global atomics bound the kernels that use it, so larger
// blocks (more particles sharing a cell) pay off.  key_of(i) >= 0; cell_count
// zeroed before the launch.
constexpr int kKeysThreads = 1024;

template <int PPT, class KeyOf>
__device__ __forceinline__ void block_ranks(int n, int *__restrict__ key, int *__restrict__ rank,
                                            int *__restrict__ cell_count, KeyOf key_of) {
    constexpr int kSlots = 2 * kKeysThreads * PPT;   // open addressing, at most half full
    constexpr int kShift = 32 - __builtin_ctz(kSlots);
    __shared__ int skey[kSlots];
    __shared__ int scnt[kSlots];
    for (int t = threadIdx.x; t < kSlots; t += blockDim.x) {
        skey[t] = -1;
        scnt[t] = 0;
    }
    __syncthreads();
    int slot[PPT], local[PPT];
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
        const long long i = ((long long)blockIdx.x * PPT + p) * kKeysThreads + threadIdx.x;
        slot[p] = -1;
        local[p] = 0;
        if (i < n) {
            const int k = key_of((size_t)i);
            key[i] = k;
            // k >= 0 and the table never fills, so the probe ends
            int sl = (int)(((unsigned)k * 2654435761u) >> kShift);
            for (;;) {
                const int old = atomicCAS(&skey[sl], -1, k);
                if (old == -1 || old == k) break;
                sl = (sl + 1) & (kSlots - 1);
            }
            slot[p] = sl;
            local[p] = atomicAdd(&scnt[sl], 1);
        }
    }
    __syncthreads();
    // one global atomic per occupied slot; its base replaces the count
    for (int t = threadIdx.x; t < kSlots; t += blockDim.x) {
        const int kk = skey[t];
        if (kk >= 0) scnt[t] = atomicAdd(&cell_count[kk], scnt[t]);
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
        const long long i = ((long long)blockIdx.x * PPT + p) * kKeysThreads + threadIdx.x;
        if (slot[p] >= 0) rank[i] = scnt[slot[p]] + local[p];
    }
}

// Particles per thread: the largest block (more particles per global atomic)
// that still gives every CU one, 8 from N = 2^21, 1 below 2^19.
inline int keys_per_thread(int n) {
    const size_t per_cu = (size_t)n / (256 * kKeysThreads);
    return per_cu >= 8 ? 8 : per_cu >= 4 ? 4 : per_cu >= 2 ? 2 : 1;
}

// ---- launchers (host functions defined in the .hip files) -----------------

// sort.hip
hipError_t launch_fill_i32(int *p, int v, size_t n, hipStream_t s);
hipError_t launch_fill_f64(double *p, double v, size_t n, hipStream_t s);
// cell key and rank inside the cell of every particle (cell_count and *done
// zeroed); where keys_scan_cells(cells), cell_count is also scanned, as
// launch_scan1 leaves it
bool keys_scan_cells(size_t ncells);
hipError_t launch_keys(const double *pos, int n, const Geom &g, int *key, int *rank,
                       int *cell_count, int *done, hipStream_t s);
size_t scan_block_sums_needed(size_t n);
// exclusive scan of n int32 values; out has n+1 entries (out[n] = total).
// in may equal out.
hipError_t launch_scan(const int *in, int *out, size_t n, int *block_sums, hipStream_t s);
// the same in one launch (decoupled look-back) for up to 64 tiles of
// kScanTile values, else as launch_scan (with bsum): status holds
// scan1_status_needed(n) entries and *ctr one int, both zeroed before the
// launch; a look-back that waited past its poll limit raises *stall
size_t scan1_status_needed(size_t n);
hipError_t launch_scan1(const int *in, int *out, size_t n, unsigned long long *status, int *ctr,
                        unsigned long long *stall, int *bsum, hipStream_t s);
// scatter into tile -> subtile order: particles of subtiles that the fine
// order leaves as they are (at most max(csize, kFineMin)) go to sp2/perm2/sel2,
// the others to sp/perm/sel_s for launch_fine_order; the subtiles above
// kFineBig particles are listed in big_list (1 + n / kFineBig ints,
// big_list[0] zeroed before the launch)
// stable: ranks from launch_stable_ranks (already in fine order), so every
// subtile goes to sp2/perm2/sel2 and no fine-order pass follows
hipError_t launch_scatter(const double *pos, const double *mass, const uint8_t *sel, int n,
                          const Geom &g, const int *key, const int *rank,
                          const int *cell_start, int fp32, int csize, bool stable, double4 *sp,
                          int *perm, uint8_t *sel_s, double4 *sp2, int *perm2, uint8_t *sel2,
                          int *big_list, hipStream_t s);
// Deterministic mode: rank[i] = place of particle i in its cell when the
// cell's particles are ordered by (fine sub-cell, index) (cell_start: the
// scanned cell counts; key: launch_keys' cell keys).  Scratch: k64a/k64b n
// each, va/vb n each, hist stable_rank_hist_ints(n) + 1, bsum for a scan of
// that many values.
size_t stable_rank_hist_ints(int n);
hipError_t launch_stable_ranks(const double *pos, int n, const Geom &g, const int *key,
                               const int *cell_start, unsigned long long *k64a,
                               unsigned long long *k64b, int *va, int *vb, int *hist, int *bsum,
                               int *rank, hipStream_t s);
// Deterministic mode: the sums of clusters with several items from the
// items' partial slots (partials[(item * csize + receiver) * 3 + c]), added
// in item order into out (item_off: the scanned item counts per cluster)
hipError_t launch_item_reduce(const Cluster *clusters, const int *n_clusters_dev, int bound,
                              const int *item_off, const double *partials, int csize,
                              const int *rperm, double *out, long long out_stride,
                              hipStream_t s);
// reorder the particles of every subtile by the Morton index of their fine
// sub-cell (sp/perm/sel -> sp2/perm2/sel2; sel == nullptr: no selector;
// fkey/frank: n ints of scratch; big_list from launch_scatter)
hipError_t launch_fine_order(const double4 *sp, const int *perm, const uint8_t *sel,
                             const int *cell_start, const Geom &g, int *fkey, int *frank,
                             double4 *sp2, int *perm2, uint8_t *sel2, int n, int csize,
                             const int *big_list, hipStream_t s);
// Receivers of every subset compacted in one launch: prefix[k n + p] (n_sub n
// + 1 ints) = receivers before particle p of subset k, and the receivers'
// records and original indices in rp / rperm at those places.  status:
// receivers_status_needed(n_sub n) entries and *ctr zeroed before the launch.
size_t receivers_status_needed(size_t rows);
hipError_t launch_receivers(const uint8_t *sel_s, int n, int n_sub, int kind,
                            const uint8_t *thr_host, const double4 *sp, const int *perm,
                            int *prefix, double4 *rp, int *rperm, unsigned long long *status,
                            int *ctr, unsigned long long *stall, hipStream_t s);
// Clusters and work items of a call in one launch.
struct PlanArgs {
    const int *cell_start;
    const int *prefix;      // of launch_receivers; nullptr: every particle a receiver
    int n, n_sub, csize, target, half;
    int split;              // dense tiles of one subtile into runs of about this many records (0: not)
    Cluster *clusters;      // tile, subset, begin and count of every cluster
    Item *items;            // nullptr: counted only
    int *item_off;          // nullptr, or the first item of every cluster (and the total)
    unsigned long long *status;   // plan_status_needed() entries, zeroed
    int *ctr;                     // zeroed
    unsigned long long *stall;
    int *n_clusters, *n_items;    // totals on the device
    int *host_tot;          // pinned: receivers, clusters and items
};
size_t plan_status_needed(int n_sub, const Geom &g);
hipError_t launch_plan(const PlanArgs &p, const Geom &g, hipStream_t s);
// every cluster's items at their offsets item_off of launch_plan (for arrays
// sized after the count is known); at most `bound` clusters
hipError_t launch_item_write(const Cluster *clusters, const int *n_clusters_dev, int bound,
                             const int *cell_start, const Geom &g, int target, int half, int split,
                             const int *item_off, Item *items, hipStream_t s);
// 32-bin histogram of particles per tile (log2 bins; bin 0: empty tiles),
// the occupancy signature the autotuner files its results under
hipError_t launch_tile_hist(const int *cell_start, const Geom &g, int *hist32, hipStream_t s);
// the bounding box of every cluster from its receivers rp (indexed like the
// clusters' begin); *n_clusters_dev clusters, at most `bound`.  w != nullptr
// (the adjoint, every particle a receiver): also wa[p] = the weight of sorted
// particle p (0 where sel is given and 0; FP32 records for fp32 calls)
hipError_t launch_cluster_finish(Cluster *clusters, const int *n_clusters_dev, size_t bound,
                                 int csize, const double4 *rp, const double *w,
                                 const uint8_t *sel, const int *perm, int fp32, double4 *wa,
                                 hipStream_t s);
// up to kFillMax int regions set to their values in one launch
constexpr int kFillMax = 8;
struct FillSet {
    int *p[kFillMax];
    size_t n[kFillMax];
    int v[kFillMax];
    int first[kFillMax + 1];   // set by launch_fill_multi
    int count;
    void add(int *ptr, size_t len, int val) {
        p[count] = ptr;
        n[count] = len;
        v[count] = val;
        ++count;
    }
};
hipError_t launch_fill_multi(FillSet f, hipStream_t s);

// force.hip
enum PairMode { FWD_F32 = 0, FWD_F64 = 1, BWD_F32 = 2, BWD_F64 = 3 };
constexpr int kXcds = 8;   // MI355X: workgroups are dealt round-robin to 8 XCDs
static_assert(kCounterCopies == kXcds, "one Counters copy per XCD");
// ints between the XCD work counters: each in a 256 B line of its own, so
// claims from different XCDs do not queue on one cache line
constexpr int kQueueStride = 64;

struct PairArgs {
    const double4 *sp;       // suppliers in sorted order
    const double4 *rp;       // receivers
    const int *cell_start;
    const Cluster *clusters;
    const Item *items;
    const double4 *wa;       // backward: w * [active] of the sorted particles (FP32: float4 bits)
    int *queue;              // kXcds work counters kQueueStride ints apart, zero at launch
    const int *rperm;        // original index of each receiver row (indexed like rp)
    double *out;             // n_sub x n x 3, zeroed before the launch
    long long out_stride;    // elements per subset in out (3 n)
    Counters *counters;      // kCounterCopies copies, kCounterStride apart
    // the item count, read on the device (the host need not wait for it)
    const int *n_items_dev;
    int unit_mass;           // no mass array: every mu_j is 1 (forward kernels specialise)
    int csize;               // cluster size (receivers per cluster, 8..64)
    // tabulated FP32 forward shape (kernel kind 1 or 2, see force.hip)
    const float *htab;       // NGP: tab_n values; linear: tab_n (value, slope) pairs
    float tab_scale;         // table entries per unit of r^2: tab_n / r_cut^2
    int tab_n;
    // mutual kernel: FP32 r^2 in [rc2_lo, rc2_hi) is tested again in FP64
    float rc2_lo, rc2_hi;
    // deterministic mode: items of clusters with several items store their
    // sums in partial slots ((item * csize + receiver) * 3) instead of
    // adding them with atomics (nullptr: atomics)
    double *partials;
    Geom g;
};

constexpr int kTabFloats = 4096;   // LDS floats a table may take (16 KB)
enum ShapeKind { SHAPE_POLY = 0, SHAPE_TAB_NGP = 1, SHAPE_TAB_LINEAR = 2 };
// Fills the table of H(t) (g(u) / r^3 = r^-3 + H(t) / (2 x_s)^3, t = u^2) on
// r^2 in [0, rc2): NGP holds H at the n bin centres, linear the value at the
// n + 1 nodes as (value, next - value) pairs.
hipError_t launch_build_htab(int kind, int n, const Geom &g, float *tab, hipStream_t s);
// screen != 0: every supplier is tested against the cluster's box first and
// the survivors (with the adjoint's weights) stream from LDS
// tab: ShapeKind of the FP32 forward shape (the other modes ignore it)
hipError_t launch_pairs(int mode, int screen, int tab, const PairArgs &a, int grid,
                        hipStream_t s);

// Long-range PM (pm.hip).  real: n^3 FP64 (rho, then phi), x fastest;
// spec: n^2 rows of n/2 + 1 complex FP64 (kx fastest) at a stride rounded up
// to 8; tw: n/2 twiddles; w1, k2:
// per-axis kernel tables of n values; scale = 4 pi / h^4 / n^3.
struct PmArgs {
    int n;
    double *real;
    double2 *spec;
    const double2 *tw;
    const double *w1, *k2;
    double scale;
};
// The particles are sorted by bins of kPmBin^3 lower CIC nodes.  bins: an int
// array of pm_sort_ints(n, n_part) entries (16-byte aligned) for the bins'
// counts, scanned in place into the first sorted index of each bin, and the
// sort's small counters and lists.
constexpr int kPmBin = 8;
struct PmSort {
    int *start;                   // (n / kPmBin)^3 + 1
    int *over;                    // runs of dense bins: their number, then (bin, first) pairs
    unsigned long long *status;   // the scan's look-back words
    unsigned long long *stall;    // not in the array: set by the caller
    int *ctr;
    size_t ints;                  // the array's length
};
PmSort pm_sort_layout(int *bins, int n, int n_part);
// twiddles, kernel tables, and the cleared sort array
hipError_t launch_pm_prepare(int n, double box, double x_s, double2 *tw, double *w1, double *k2,
                             const PmSort &ps, hipStream_t s);
// key/rank: n_part ints of scratch; bsum: scan block sums; rec (CIC fractions,
// mu), nkey (the lower node) and perm (the particle, ~particle where it
// receives nothing) n_part entries in bin order
hipError_t launch_pm_sort(const double *pos, const double *mass, const uint8_t *active,
                          int n_part, int n, double box, double h, int *key, int *rank,
                          const PmSort &ps, int *bsum, double4 *rec, int *nkey, int *perm,
                          hipStream_t s);
// rho (n^3, fully written) from the sorted records
hipError_t launch_pm_deposit(const double4 *rec, const int *nkey, const PmSort &ps, int n_part,
                             double *rho, int n, hipStream_t s);
// ev (optional): 4 events recorded after the x, y and z passes and the y
// inverse pass
hipError_t launch_pm_fft_chain(const PmArgs &a, hipStream_t s, hipEvent_t *ev);
hipError_t launch_pm_readout(const double4 *rec, const int *nkey, const int *perm, int n_part,
                             const double *phi, int n, double *acc, hipStream_t s);
// pair-kernel workgroups resident per CU for the variant launch_pairs would run
int pairs_blocks_per_cu(int mode, int screen, int tab, int csize, int unit_mass, int soft);
// All-active FP32 forward (bwd: the FP32 adjoint, every particle a receiver,
// weights in a.wa; f64: the FP64 kinds, the adjoint without softening) with each pair
// evaluated once for both partners (clusters
// of csize = 16, 32 or 64 receivers, items over the upper half of the
// stencil).  a.out: three FP64 arrays of a.out_stride = n sums in sorted
// order, zeroed before the launch; launch_mutual_out then writes acc_out.
hipError_t launch_pairs_mutual(const PairArgs &a, bool bwd, bool f64, int grid, hipStream_t s);
int mutual_blocks_per_cu(int csize, int unit_mass, bool bwd, bool soft, bool f64);
hipError_t launch_mutual_out(const double *sums, const int *perm, int n, double *out,
                             hipStream_t s);

// KDK step (kdk.hip).  Times in units of tau / 2, tau = dt / 2^L.
struct KdkArgs {
    double dt;
    double two_eta_eps;   // 2 eta eps of eq. rung
    double half_tau;
    int L;                // highest rung of the period
    int period;           // n_steps 2^(L+1)
    int max_rung;
    int fixed;            // 1: rungs are inputs and never change
};
// census (9 ints, zeroed): particles per rung 0 .. 7, and the highest rung
hipError_t launch_kdk_assign(const double *acc, int n, const KdkArgs &k, uint8_t *rung,
                             int *census, hipStream_t s);
hipError_t launch_kdk_first(double *vel, const double *acc, int n, const KdkArgs &k,
                            const uint8_t *rung, int *t_q, int *t_next, hipStream_t s);
struct KdkAdvance {
    double *pos, *vel;
    const double *acc;
    uint8_t *due, *rung;
    int *t_q, *t_next;
    int n;
    double tau, box;
    const Counters *counters;        // of the force call before a kick
    unsigned long long *pairs;       // the period's accepted pairs
};
// kick: the particles due at t; drift: over tau to t + 2, the particles due
// there marked and counted in *n_due (zeroed)
hipError_t launch_kdk_advance(const KdkAdvance &a, bool kick, bool drift, int t, const KdkArgs &k,
                              int *n_due, hipStream_t s);
// vel += dk acc over n x 3 values
hipError_t launch_axpy3(double *vel, const double *acc, int n, double dk, hipStream_t s);
hipError_t launch_kdk_accum(const Counters *c, unsigned long long *total, hipStream_t s);

}  // namespace p3m
