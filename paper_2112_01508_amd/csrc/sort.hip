// Tile/subtile counting sort, receiver compaction and work-item planning.
//
// Section 2.1.3 ("Tiles", "Subtiles", "Other optimisations"): particles are
// sorted in O(N) into tiles of side >= r_cut, each split into ns^3
// subtiles, and stored in tile -> subtile -> particle order.  On the GPU the
// sort is a counting sort over the fine cells (histogram with atomics ->
// exclusive scan -> scatter).  Receivers (the particles on active rungs,
// section 2.2.2) are compacted per tile and grouped into clusters of at most
// one wavefront; each cluster is then split into work items over its 27
// neighbour tiles so that one persistent launch can balance the very uneven
// work of clustered particle sets.
#include "p3msr_internal.hpp"

#include <algorithm>
#include <climits>

namespace p3m {

namespace {

__global__ void k_fill_i32(int *p, int v, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    if (((uintptr_t)p & 15) == 0) {
        // 16-byte stores for the bulk, then the tail
        int4 *p4 = reinterpret_cast<int4 *>(p);
        const size_t n4 = n / 4;
        const int4 v4 = make_int4(v, v, v, v);
        for (size_t j = i; j < n4; j += stride) p4[j] = v4;
        for (size_t j = 4 * n4 + i; j < n; j += stride) p[j] = v;
        return;
    }
    for (; i < n; i += stride) p[i] = v;
}

__global__ void k_fill_f64(double *p, double v, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

// Position wrapped into [0, box).
__device__ inline double wrap_coord(double x, const Geom &g) {
    double w = x - g.box * floor(x * g.inv_box);
    if (!(w < g.box)) w = 0.0;   // rounding up to box, or NaN
    if (w < 0.0) w = 0.0;
    return w;
}

__device__ inline int cell_of(double w, const Geom &g) {
    int c = (int)(w * g.inv_cell);
    return c < 0 ? 0 : (c >= g.nc ? g.nc - 1 : c);
}

__device__ inline int key_of(int cx, int cy, int cz, const Geom &g) {
    int tx = cx / g.ns, ty = cy / g.ns, tz = cz / g.ns;
    int sx = cx - tx * g.ns, sy = cy - ty * g.ns, sz = cz - tz * g.ns;
    int tile = (tx * g.nt + ty) * g.nt + tz;
    return tile * g.ns3 + (sx * g.ns + sy) * g.ns + sz;
}

__device__ inline int block_exclusive_scan(int v, int *lds, int *total) {
    // wave-level inclusive scan with shuffles, then across the block's waves
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    int x = v;
    for (int off = 1; off < kWave; off <<= 1) {
        int y = __shfl_up(x, off, kWave);
        if (lane >= off) x += y;
    }
    if (lane == kWave - 1) lds[wave] = x;
    __syncthreads();
    const int nw = blockDim.x / kWave;
    int base = 0, all = 0;
    for (int w = 0; w < nw; ++w) {
        int s = lds[w];
        if (w < wave) base += s;
        all += s;
    }
    __syncthreads();
    *total = all;
    return base + x - v;
}

// Cell key and rank inside the cell of every particle.  n_scan != 0 (at most
// kKeysScan cells): the block that finishes last scans the counts too, in place
// (cell_count[n_scan] = n), which saves the launch of one to eight blocks (a
// call on 4096 particles 46.6 -> 43.1 us, on 32768 73.6 -> 69.8 us).  Every
// block has its atomics' results before it draws from *done (zeroed before the
// launch), and the last one reads the counts with device-scope loads.
constexpr int kKeysScan = 4 * kKeysThreads;

template <int PPT>
__global__ __launch_bounds__(kKeysThreads) void k_keys(const double *__restrict__ pos, int n,
                                                       Geom g, int *__restrict__ key,
                                                       int *__restrict__ rank, int *cell_count,
                                                       int n_scan, int *done) {
    block_ranks<PPT>(n, key, rank, cell_count, [&](size_t i) {
        const double wx = wrap_coord(pos[3 * i], g);
        const double wy = wrap_coord(pos[3 * i + 1], g);
        const double wz = wrap_coord(pos[3 * i + 2], g);
        return key_of(cell_of(wx, g), cell_of(wy, g), cell_of(wz, g), g);
    });
    if (n_scan == 0) return;
    __shared__ int lds[kKeysThreads / kWave];
    __shared__ int last;
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(done, 1) == (int)gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    int v[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int c = 4 * (int)threadIdx.x + j;
        v[j] = c < n_scan ? __hip_atomic_load(cell_count + c, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT)
                          : 0;
        sum += v[j];
    }
    int total;
    int run = block_exclusive_scan(sum, lds, &total);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int c = 4 * (int)threadIdx.x + j;
        if (c < n_scan) cell_count[c] = run;
        run += v[j];
    }
    if (threadIdx.x == 0) cell_count[n_scan] = total;
}

// ---- exclusive scan (reduce / top / down-sweep) -----------------------------

// Tiles of kScanTile values; a block's threads load them striped (value
// k * kScanBlock + t), so every wave load is coalesced.
__global__ __launch_bounds__(kScanBlock) void k_scan_reduce(const int *__restrict__ in, size_t n,
                                                            int *__restrict__ bsum) {
    __shared__ int lds[kScanBlock / kWave];
    const size_t base = (size_t)blockIdx.x * kScanTile + threadIdx.x;
    int s = 0;
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
        const size_t i = base + (size_t)k * kScanBlock;
        if (i < n) s += in[i];
    }
    int total;
    block_exclusive_scan(s, lds, &total);
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void k_scan_top(int *__restrict__ bsum, int nb,
                                                   int *__restrict__ out_total) {
    __shared__ int lds[1024 / kWave];
    int carry = 0;
    for (int base = 0; base < nb; base += 1024) {
        int i = base + threadIdx.x;
        int v = i < nb ? bsum[i] : 0;
        int total;
        int ex = block_exclusive_scan(v, lds, &total);
        if (i < nb) bsum[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) {
        bsum[nb] = carry;
        *out_total = carry;
    }
}

// Down-sweep: the tile is loaded striped into LDS, each thread scans its
// kScanPerThread consecutive values there (a pad word per 16 keeps the
// per-thread reads free of bank conflicts), and the result is stored striped.
// in and out may be the same array.
__device__ __forceinline__ int scan_pad(int i) { return i + (i >> 4); }

__global__ __launch_bounds__(kScanBlock) void k_scan_down(const int *in, int *out, size_t n,
                                                          const int *__restrict__ bsum) {
    __shared__ int lds[kScanBlock / kWave];
    __shared__ int tile[kScanTile + kScanTile / 16];
    const size_t base = (size_t)blockIdx.x * kScanTile;
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
        const int e = k * kScanBlock + threadIdx.x;
        const size_t i = base + e;
        tile[scan_pad(e)] = i < n ? in[i] : 0;
    }
    __syncthreads();
    const int first = threadIdx.x * kScanPerThread;
    int v[kScanPerThread];
    int s = 0;
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
        v[k] = tile[scan_pad(first + k)];
        s += v[k];
    }
    int total;
    int run = block_exclusive_scan(s, lds, &total) + bsum[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
        tile[scan_pad(first + k)] = run;
        run += v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
        const int e = k * kScanBlock + threadIdx.x;
        const size_t i = base + e;
        if (i < n) out[i] = tile[scan_pad(e)];
    }
}

// Decoupled look-back.  Each block takes the next tile number from a counter,
// so every tile before it belongs to a block that is already running; it
// publishes its tile's sum at once (nothing delays that), then its first wave
// reads the status of the 64 tiles before it together, adding their sums back
// to the nearest published inclusive prefix (another window of 64 if there is
// none), and publishes its own.  status[t] (zeroed before the launch): 0
// nothing yet, kBackSum | sum, or kBackPrefix | inclusive prefix, with 62 bits
// of value (one sum, or two that are packed).  A wait longer than kBackSpins
// polls (which a running predecessor cannot cause) ends the wait anyway and
// raises *stall.
constexpr unsigned long long kBackSum = 1ull << 62, kBackPrefix = 2ull << 62;
constexpr unsigned long long kBackValue = kBackSum - 1ull;
constexpr int kBackSpins = 1 << 20;

// The sum of the tiles before t (every lane of the calling wave, which all
// must take part); publishes tile t's own sum `total`.
__device__ __forceinline__ unsigned long long look_back(unsigned long long *status, int t,
                                                        unsigned long long total,
                                                        unsigned long long *stall) {
    const int lane = threadIdx.x & (kWave - 1);
    if (lane == 0)
        __hip_atomic_store(&status[t], (t == 0 ? kBackPrefix : kBackSum) | total,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long excl = 0;
    for (int top = t - 1; top >= 0; top -= kWave) {
        // tiles before 0 count as a prefix of 0, so every window that
        // reaches them ends the walk
        const int p = top - lane;
        int spins = 0;
        int near = kWave;   // lowest lane (nearest tile) holding a prefix
        unsigned long long st = 0;
        for (;;) {
            st = p >= 0 ? __hip_atomic_load(&status[p], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT)
                        : kBackPrefix;
            const unsigned long long pm = __builtin_amdgcn_ballot_w64((st >> 62) == 2);
            const unsigned long long em = __builtin_amdgcn_ballot_w64((st >> 62) == 0);
            near = pm ? __builtin_ctzll(pm) : kWave;
            const unsigned long long need = near >= kWave - 1 ? ~0ull : ((2ull << near) - 1ull);
            if ((em & need) == 0) break;
            if (++spins >= kBackSpins) {
                if (lane == 0) atomicAdd(stall, 1ull);
                near = -1;   // give up: the result is flagged as invalid
                break;
            }
        }
        if (near < 0) break;
        unsigned long long add = lane <= near ? st & kBackValue : 0ull;
        for (int off = kWave / 2; off > 0; off >>= 1) add += __shfl_xor(add, off, kWave);
        excl += add;
        if (near < kWave) break;
    }
    if (lane == 0 && t > 0)
        __hip_atomic_store(&status[t], kBackPrefix | (excl + total), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    return excl;
}

// Single-pass exclusive scan.  out[n] = the total; in may equal out.
constexpr int kScan1MaxTiles = 64;   // larger scans take the three-kernel path

__global__ __launch_bounds__(kScanBlock) void k_scan_1pass(const int *in, int *out, size_t n,
                                                           unsigned long long *status, int *ctr,
                                                           unsigned long long *stall) {
    __shared__ int lds[kScanBlock / kWave];
    __shared__ int tile[kScanTile + kScanTile / 16];
    __shared__ int s_tile, s_excl;
    if (threadIdx.x == 0) s_tile = atomicAdd(ctr, 1);
    __syncthreads();
    const int t = s_tile;
    const size_t base = (size_t)t * kScanTile;
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
        const int e = k * kScanBlock + threadIdx.x;
        const size_t i = base + e;
        tile[scan_pad(e)] = i < n ? in[i] : 0;
    }
    __syncthreads();
    const int first = threadIdx.x * kScanPerThread;
    int v[kScanPerThread];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
        v[k] = tile[scan_pad(first + k)];
        sum += v[k];
    }
    int total;
    int run = block_exclusive_scan(sum, lds, &total);
    if (threadIdx.x < kWave) {
        const int excl = (int)look_back(status, t, (unsigned)total, stall);
        if (threadIdx.x == 0) {
            s_excl = excl;
            if (base + kScanTile >= n) out[n] = excl + total;   // the last tile
        }
    }
    __syncthreads();
    run += s_excl;
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
        tile[scan_pad(first + k)] = run;
        run += v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
        const int e = k * kScanBlock + threadIdx.x;
        const size_t i = base + e;
        if (i < n) out[i] = tile[scan_pad(e)];
    }
}

// ---- scatter into tile -> subtile order --------------------------------------

// Particles of subtiles with at most keep_max particles keep their scattered
// order, so they go straight to the final arrays (sp_f, perm_f, sel_f); the
// others go to the staging arrays that the fine-order pass reorders from.
__global__ void k_scatter(const double *__restrict__ pos, const double *__restrict__ mass,
                          const uint8_t *__restrict__ sel, int n, Geom g,
                          const int *__restrict__ key, const int *__restrict__ rank,
                          const int *__restrict__ cell_start, int fp32, int keep_max,
                          double4 *__restrict__ sp_s, int *__restrict__ perm_s,
                          uint8_t *__restrict__ sel_st, double4 *__restrict__ sp_f,
                          int *__restrict__ perm_f, uint8_t *__restrict__ sel_f,
                          int *__restrict__ big_list) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int k = key[i];
    const int c0 = cell_start[k], cnt = cell_start[k + 1] - c0;
    const int q = rank[i];
    int dst = c0 + q;
    const bool direct = cnt <= keep_max;
    // the particle of rank 0 lists its subtile for the block-wide fine order
    if (q == 0 && !direct && cnt > kFineBig) big_list[1 + atomicAdd(big_list, 1)] = k;
    double4 *__restrict__ sp = direct ? sp_f : sp_s;
    int *__restrict__ perm = direct ? perm_f : perm_s;
    uint8_t *__restrict__ sel_s = direct ? sel_f : sel_st;
    double4 v;
    v.x = wrap_coord(pos[3 * (size_t)i], g);
    v.y = wrap_coord(pos[3 * (size_t)i + 1], g);
    v.z = wrap_coord(pos[3 * (size_t)i + 2], g);
    double mu = mass ? mass[i] : 1.0;
    if (fp32) {
        float mf = (float)mu;
        v.w = __longlong_as_double((long long)(unsigned int)__float_as_uint(mf));
    } else {
        v.w = mu;
    }
    sp[dst] = v;
    perm[dst] = i;
    if (sel) sel_s[dst] = sel[i];   // no selector: every particle takes part
}

// ---- fine order inside subtiles -------------------------------------------------

// Morton index of the particle's 8x8x8 sub-cell inside its subtile.
__device__ inline int fine_key(const double4 &p, const Geom &g) {
    int f[3];
    const double w[3] = {p.x, p.y, p.z};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double u = w[d] * g.inv_cell;
        int c = (int)u;
        c = c < 0 ? 0 : (c >= g.nc ? g.nc - 1 : c);
        int q = (int)((u - c) * kFineSide);
        f[d] = q < 0 ? 0 : (q >= kFineSide ? kFineSide - 1 : q);
    }
    int k = 0;
#pragma unroll
    for (int b = 0; b < 3; ++b)
        k |= (((f[0] >> b) & 1) << (3 * b + 2)) | (((f[1] >> b) & 1) << (3 * b + 1)) |
             (((f[2] >> b) & 1) << (3 * b));
    return k;
}

__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Fine order.  Inside every subtile holding more than keep_max particles the
// particles are reordered by fine_key (a counting sort over kFineBins bins in
// LDS); smaller subtiles are already in place (the scatter wrote them to
// sp2/perm2/sel2).  Reads sp/perm/sel and writes sp2/perm2/sel2 (sel ==
// nullptr: no selector); fkey/frank are scratch indexed by sorted position.
// Consecutive receivers then lie close together, so small clusters have small
// bounding boxes.
//
// The first big_blocks blocks take the subtiles above kFineBig particles
// (listed by the scatter: big_list[0] counts them, the ids follow in any
// order), one after the other with one bin per thread in the scan: a single
// wave would take the densest halo cores alone, long after the rest of the
// grid.  The other blocks take one tile per wave.  Both in one launch, so
// that the dense subtiles run beside the rest without a second stream (whose
// events cost the call 6 to 12 us each).
__global__ __launch_bounds__(kFineBins) void k_fine_order(
    const double4 *__restrict__ sp, const int *__restrict__ perm, const uint8_t *__restrict__ sel,
    const int *__restrict__ cs, Geom g, int *__restrict__ fkey, int *__restrict__ frank,
    double4 *__restrict__ sp2, int *__restrict__ perm2, uint8_t *__restrict__ sel2, int keep_max,
    int big_blocks, const int *__restrict__ big_list) {
    __shared__ int hists[kFineWaves][kFineBins];
    if ((int)blockIdx.x < big_blocks) {
        int *hist = hists[0];
        int *lds = hists[1];
        const int t = threadIdx.x;
        const int n_big = big_list[0];
        for (int j = blockIdx.x; j < n_big; j += big_blocks) {
            const int cell = big_list[1 + j];
            const int a0 = cs[cell], a1 = cs[cell + 1];
            hist[t] = 0;
            __syncthreads();
            for (int i = a0 + t; i < a1; i += kFineBins) {
                const int k = fine_key(sp[i], g);
                fkey[i] = k;
                frank[i] = atomicAdd(&hist[k], 1);
            }
            __syncthreads();
            int total;
            const int ex = block_exclusive_scan(hist[t], lds, &total);
            hist[t] = ex;   // every thread has read its own bin in the call above
            __syncthreads();
            for (int i = a0 + t; i < a1; i += kFineBins) {
                const int dst = a0 + hist[fkey[i]] + frank[i];
                sp2[dst] = sp[i];
                perm2[dst] = perm[i];
                if (sel) sel2[dst] = sel[i];
            }
            __syncthreads();
        }
        return;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    int *hist = hists[w];
    const long long stride = (long long)(gridDim.x - big_blocks) * kFineWaves;
    for (long long tile = (long long)(blockIdx.x - big_blocks) * kFineWaves + w; tile < g.nt3;
         tile += stride) {
        const int *c = cs + tile * g.ns3;
        for (int s = 0; s < g.ns3; ++s) {
            const int a0 = c[s], a1 = c[s + 1];
            if (a1 - a0 <= keep_max || a1 - a0 > kFineBig) continue;
            for (int b = lane; b < kFineBins; b += kWave) hist[b] = 0;
            wave_lds_sync();
            for (int i = a0 + lane; i < a1; i += kWave) {
                const int k = fine_key(sp[i], g);
                fkey[i] = k;
                frank[i] = atomicAdd(&hist[k], 1);
            }
            wave_lds_sync();
            // exclusive scan of the bins: lane l owns bins [l*P, l*P + P)
            constexpr int P = kFineBins / kWave;
            int v[P], sum = 0;
#pragma unroll
            for (int q = 0; q < P; ++q) {
                v[q] = hist[lane * P + q];
                sum += v[q];
            }
            int incl = sum;
            for (int off = 1; off < kWave; off <<= 1) {
                const int y = __shfl_up(incl, off, kWave);
                if (lane >= off) incl += y;
            }
            int run = incl - sum;
#pragma unroll
            for (int q = 0; q < P; ++q) {
                hist[lane * P + q] = run;
                run += v[q];
            }
            wave_lds_sync();
            for (int i = a0 + lane; i < a1; i += kWave) {
                const int dst = a0 + hist[fkey[i]] + frank[i];
                sp2[dst] = sp[i];
                perm2[dst] = perm[i];
                if (sel) sel2[dst] = sel[i];
            }
            wave_lds_sync();
        }
    }
}

// ---- stable order (deterministic mode) ----------------------------------------
//
// The counting sort above ranks the particles of a cell (and of a fine
// sub-cell) by atomics, so their order inside a cell can change between
// calls, and with it the order of every floating-point sum.  The stable path
// sorts the composite key cell << kFineBits | fine sub-cell with an LSD radix
// sort (8-bit digits, stable passes) carrying the particle index; a cell's
// particles then come in (fine sub-cell, index) order, the same on every call,
// and the scatter writes that order directly (no fine-order pass).

constexpr int kFineBits = 9;
static_assert(kFineBins == 1 << kFineBits, "fine sub-cells per subtile");
constexpr int kRsTile = 2048;   // elements per block (one wave) of a radix pass

__global__ void k_rs_keys(const double *__restrict__ pos, int n, Geom g,
                          const int *__restrict__ key, unsigned long long *__restrict__ k64,
                          int *__restrict__ val) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double4 p;
    p.x = wrap_coord(pos[3 * (size_t)i], g);
    p.y = wrap_coord(pos[3 * (size_t)i + 1], g);
    p.z = wrap_coord(pos[3 * (size_t)i + 2], g);
    p.w = 0.0;
    k64[i] = ((unsigned long long)(unsigned)key[i] << kFineBits) | (unsigned)fine_key(p, g);
    val[i] = i;
}

// Digit counts of one block's elements, digit-major (hist[d * nblk + b]), so
// that the exclusive scan of hist gives every (digit, block) its first slot.
__global__ __launch_bounds__(kWave) void k_rs_hist(const unsigned long long *__restrict__ k64,
                                                   int n, int shift, int nblk,
                                                   int *__restrict__ hist) {
    __shared__ int cnt[256];
    const int lane = threadIdx.x;
    for (int d = lane; d < 256; d += kWave) cnt[d] = 0;
    wave_lds_sync();
    const size_t base = (size_t)blockIdx.x * kRsTile;
    for (int k = lane; k < kRsTile; k += kWave) {
        const size_t e = base + k;
        if (e < (size_t)n) atomicAdd(&cnt[(int)((k64[e] >> shift) & 255u)], 1);
    }
    wave_lds_sync();
    for (int d = lane; d < 256; d += kWave) hist[(size_t)d * nblk + blockIdx.x] = cnt[d];
}

// Stable scatter of one block's elements by digit: 64 elements at a time in
// index order, each placed after the block's earlier elements of its digit
// (the running slot in LDS) and after the lanes below it with the same digit
// (the lanes whose eight digit-bit ballots all agree with its own).
__global__ __launch_bounds__(kWave) void k_rs_scatter(
    const unsigned long long *__restrict__ kin, const int *__restrict__ vin, int n, int shift,
    int nblk, const int *__restrict__ off, unsigned long long *__restrict__ kout,
    int *__restrict__ vout) {
    __shared__ int run[256];
    const int lane = threadIdx.x;
    for (int d = lane; d < 256; d += kWave) run[d] = off[(size_t)d * nblk + blockIdx.x];
    wave_lds_sync();
    const size_t base = (size_t)blockIdx.x * kRsTile;
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int k = 0; k < kRsTile; k += kWave) {
        const size_t e = base + k + lane;
        const bool live = e < (size_t)n;
        const unsigned long long key = live ? kin[e] : 0ull;
        const int v = live ? vin[e] : 0;
        const int d = (int)((key >> shift) & 255u);
        unsigned long long m = __builtin_amdgcn_ballot_w64(live);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1;
            const unsigned long long bb = __builtin_amdgcn_ballot_w64(bit);
            m &= bit ? bb : ~bb;
        }
        const int dst = run[d] + __builtin_popcountll(m & below);
        wave_lds_sync();   // every lane has read its digit's slot
        if (live) {
            kout[dst] = key;
            vout[dst] = v;
            if ((m >> lane) == 1ull) run[d] = dst + 1;   // the group's last lane
        }
        wave_lds_sync();
    }
}

// rank[i] = place of particle i inside its cell in the stable order.
__global__ void k_rs_rank(const unsigned long long *__restrict__ k64,
                          const int *__restrict__ val, int n, const int *__restrict__ cell_start,
                          int *__restrict__ rank) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    rank[val[p]] = p - cell_start[(int)(k64[p] >> kFineBits)];
}

// ---- receiver selection and compaction ---------------------------------------

struct Thresholds { uint8_t t[64]; };

// Compaction of the receivers, subset-major in sorted order, in one pass over
// the (subset, particle) rows: tiles of kRecvTile rows, 256 ballots of
// 64 consecutive rows each; the ballots' counts are scanned over the block and
// a look-back gives the receivers of the tiles before.  prefix[row] = the
// receivers before the row (prefix[rows] the total); the receivers' records
// and original indices are gathered at their places.  (Flags, a scan of three
// kernels over them, the compaction and the gather were six launches.)
constexpr int kRecvThreads = 1024;
constexpr int kRecvPer = 16;   // rows per thread
constexpr int kRecvTile = kRecvThreads * kRecvPer;
constexpr int kRecvWaves = kRecvThreads / kWave;

__global__ __launch_bounds__(kRecvThreads) void k_receivers(
    const uint8_t *__restrict__ sel_s, int n, int n_sub, int kind, Thresholds thr,
    const double4 *__restrict__ sp, const int *__restrict__ perm, int *__restrict__ prefix,
    double4 *__restrict__ rp, int *__restrict__ rperm, unsigned long long *status, int *ctr,
    unsigned long long *stall) {
    __shared__ int cnt[kRecvPer * kRecvWaves];
    __shared__ int lds[kRecvWaves];
    __shared__ int s_tile, s_excl;
    if (threadIdx.x == 0) s_tile = atomicAdd(ctr, 1);
    __syncthreads();
    const int tile = s_tile;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const size_t rows = (size_t)n * n_sub;
    const size_t first = (size_t)tile * kRecvTile + threadIdx.x;
    const int k0 = (int)(first / n), p0 = (int)(first - (size_t)k0 * n);
    unsigned flag = 0;
    int k = k0, p = p0;
#pragma unroll
    for (int j = 0; j < kRecvPer; ++j) {
        bool f = false;
        if (first + (size_t)j * kRecvThreads < rows)
            f = kind == SEL_MASK ? sel_s[p] != 0 : sel_s[p] >= thr.t[k];
        flag |= (unsigned)f << j;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(f);
        if (lane == 0) cnt[j * kRecvWaves + wave] = __builtin_popcountll(m);
        for (p += kRecvThreads; p >= n; p -= n) ++k;
    }
    __syncthreads();
    const int v = threadIdx.x < kRecvPer * kRecvWaves ? cnt[threadIdx.x] : 0;
    int total;
    const int ex = block_exclusive_scan(v, lds, &total);
    if (wave == 0) {
        const int excl = (int)look_back(status, tile, (unsigned)total, stall);
        if (lane == 0) {
            s_excl = excl;
            if ((size_t)(tile + 1) * kRecvTile >= rows) prefix[rows] = excl + total;
        }
    }
    __syncthreads();
    if (threadIdx.x < kRecvPer * kRecvWaves) cnt[threadIdx.x] = s_excl + ex;
    __syncthreads();
    k = k0;
    p = p0;
#pragma unroll
    for (int j = 0; j < kRecvPer; ++j) {
        const bool f = (flag >> j) & 1u;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(f);
        const size_t row = first + (size_t)j * kRecvThreads;
        if (row < rows) {
            const int at = cnt[j * kRecvWaves + wave] +
                           __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            prefix[row] = at;
            if (f) {
                rp[at] = sp[p];
                rperm[at] = perm[p];
            }
        }
        for (p += kRecvThreads; p >= n; p -= n) ++k;
    }
}

// ---- clusters and work items -----------------------------------------------------

// Clusters and items of PT (subset, tile) entries per block, in one
// launch: a cluster is a run of at most csize consecutive receivers of one
// tile, so the clusters follow from the tiles' receiver counts, and a
// cluster's items from those and the particle counts of its stencil.  The
// block counts its clusters (one thread per entry) and their items (one thread
// per cluster, 256 at a time), a look-back over the blocks gives the clusters
// and items before its own (both counts packed in one status word), and the
// records are written where they belong: in entry order, as the XCD chunks of
// the item queue want them.  Counting, scanning and writing clusters and items
// in launches of their own took six, at 5 to 12 us each for sets of any size
// below 2^20 particles.
//
// The look-back chain grows with the blocks (64 predecessors per step), the
// serial work of a block with its entries: PT = 64 entries up to 2^14 of them
// (256 blocks), 512 entries beyond.
constexpr int kPlanThreads = 256;
constexpr int kPlanThreadsBig = 512;
constexpr long long kPlanBigFrom = 1 << 14;
constexpr int kPlanCache = 1024;   // item counts kept from the first pass
constexpr unsigned kPlanBits = 31;

template <bool HALF, int PT, int NT>
__global__ __launch_bounds__(NT) void k_plan(PlanArgs a, Geom g) {
    __shared__ int lds[NT / kWave];
    __shared__ int pre[PT], beg[PT], num[PT];
    __shared__ unsigned short cache[kPlanCache];
    __shared__ int s_tile, s_cl, s_it;
    const int t = threadIdx.x;
    if (t == 0) s_tile = atomicAdd(a.ctr, 1);
    __syncthreads();
    const int blk = s_tile;
    const long long entries = (long long)a.n_sub * g.nt3;
    const long long e0 = (long long)blk * PT;
    int ncl = 0;
    if (t < PT && e0 + t < entries) {
        const int k = (int)((e0 + t) / g.nt3);
        const int tile = (int)(e0 + t - (long long)k * g.nt3);
        int r0 = a.cell_start[(size_t)tile * g.ns3], r1 = a.cell_start[(size_t)(tile + 1) * g.ns3];
        if (a.prefix) {
            const size_t off = (size_t)k * a.n;
            r0 = a.prefix[off + r0];
            r1 = a.prefix[off + r1];
        }
        beg[t] = r0;
        num[t] = r1 - r0;
        ncl = (r1 - r0 + a.csize - 1) / a.csize;
    }
    int n_cl;
    const int ex = block_exclusive_scan(ncl, lds, &n_cl);
    if (t < PT) pre[t] = ex;
    __syncthreads();
    // cluster c of the block: its entry is the last with pre <= c
    auto locate = [&](int c, Cluster &cl) {
        int lo = 0, hi = PT;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= c) lo = mid;
            else hi = mid;
        }
        const int skip = (c - pre[lo]) * a.csize;
        cl.subset = (int)((e0 + lo) / g.nt3);
        cl.tile = (int)(e0 + lo - (long long)cl.subset * g.nt3);
        cl.begin = beg[lo] + skip;
        cl.count = min(a.csize, num[lo] - skip);
    };
    auto nothing = [](int, int, int, int, int, int) {};
    // the first NT clusters' stencils and item counts stay in registers
    Cluster cl1{};
    int w1[27];
    int k1 = 0;
    if (t < n_cl) {
        locate(t, cl1);
        plan_weights<HALF>(cl1.tile, cl1.begin + cl1.count, a.cell_start, g, w1);
        k1 = plan_items<HALF>(w1, a.target, g.ns3, a.split, nothing);
    }
    int mine = k1;
    for (int c = NT + t; c < n_cl; c += NT) {
        Cluster cl;
        locate(c, cl);
        int w[27];
        plan_weights<HALF>(cl.tile, cl.begin + cl.count, a.cell_start, g, w);
        const int k = plan_items<HALF>(w, a.target, g.ns3, a.split, nothing);
        if (c < kPlanCache) cache[c] = (unsigned short)min(k, 0xffff);
        mine += k;
    }
    int n_it;
    (void)block_exclusive_scan(mine, lds, &n_it);
    if (t < kWave) {
        const unsigned long long excl = look_back(
            a.status, blk, (unsigned long long)n_cl << kPlanBits | (unsigned)n_it, a.stall);
        if (t == 0) {
            s_cl = (int)(excl >> kPlanBits);
            s_it = (int)(excl & ((1u << kPlanBits) - 1u));
            if (e0 + PT >= entries) {   // the last block
                const int all_cl = s_cl + n_cl, all_it = s_it + n_it;
                *a.n_clusters = all_cl;
                *a.n_items = all_it;
                if (a.item_off) a.item_off[all_cl] = all_it;
                a.host_tot[0] = a.prefix ? a.prefix[(size_t)a.n * a.n_sub] : a.n;
                a.host_tot[1] = all_cl;
                a.host_tot[2] = all_it;
            }
        }
    }
    __syncthreads();
    const int cl0 = s_cl;
    int it0 = s_it;
    for (int c0 = 0; c0 < n_cl; c0 += NT) {
        const int c = c0 + t;
        if (c0 > 0 && c < n_cl) {
            locate(c, cl1);
            plan_weights<HALF>(cl1.tile, cl1.begin + cl1.count, a.cell_start, g, w1);
            k1 = c < kPlanCache ? cache[c] : 0xffff;
            if (k1 == 0xffff) k1 = plan_items<HALF>(w1, a.target, g.ns3, a.split, nothing);
        }
        const int k = c < n_cl ? k1 : 0;
        if (c < n_cl)
            *reinterpret_cast<int4 *>(a.clusters + cl0 + c) =
                make_int4(cl1.tile, cl1.subset, cl1.begin, cl1.count);
        int total;
        const int off = it0 + block_exclusive_scan(k, lds, &total);
        if (c < n_cl) {
            if (a.item_off) a.item_off[cl0 + c] = off;
            if (a.items) {
                const int sole = k == 1 ? kItemSole : 0;
                Item *out = a.items + off;
                plan_items<HALF>(w1, a.target, g.ns3, a.split,
                                 [&](int q, int t0, int t1, int s0, int s1, int part) {
                                     *reinterpret_cast<int4 *>(out + q) =
                                         make_int4(cl0 + c, t0 | (t1 << 8), s0 | (s1 << 16),
                                                   sole | part | (q == 0 ? kItemFirst : 0));
                                 });
            }
        }
        it0 += total;
    }
}

// Items of every cluster at their offsets; the cluster count is read on the
// device.
template <bool HALF>
__global__ void k_item_write(const Cluster *__restrict__ clusters, const int *__restrict__ n_cl,
                             const int *__restrict__ cs, Geom g, int target, int split,
                             const int *__restrict__ item_off, Item *__restrict__ items) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= *n_cl) return;
    const int off = item_off[c];
    const int sole = item_off[c + 1] - off == 1 ? kItemSole : 0;
    const Cluster &cl = clusters[c];
    int w[27];
    plan_weights<HALF>(cl.tile, cl.begin + cl.count, cs, g, w);
    plan_items<HALF>(w, target, g.ns3, split,
                     [&](int q, int t0, int t1, int s0, int s1, int part) {
                         *reinterpret_cast<int4 *>(items + off + q) =
                             make_int4(c, t0 | (t1 << 8), s0 | (s1 << 16),
                                       sole | part | (q == 0 ? kItemFirst : 0));
                     });
}

// Deterministic mode: the sums of every cluster with several items, added
// in item order from the items' partial slots (3 doubles per item and
// receiver slot); a cluster's only item stored its sums itself.
__global__ __launch_bounds__(kWave) void k_item_reduce(
    const Cluster *__restrict__ clusters, const int *__restrict__ n_cl,
    const int *__restrict__ item_off, const double *__restrict__ partials, int csize,
    const int *__restrict__ rperm, double *__restrict__ out, long long out_stride) {
    const int nc = *n_cl;
    const int r = threadIdx.x;
    for (int c = blockIdx.x; c < nc; c += gridDim.x) {
        const int i0 = item_off[c], i1 = item_off[c + 1];
        if (i1 - i0 <= 1) continue;
        const Cluster cl = clusters[c];
        if (r >= cl.count) continue;
        double sx = 0.0, sy = 0.0, sz = 0.0;
        for (int it = i0; it < i1; ++it) {
            const double *q = partials + ((size_t)it * csize + r) * 3;
            sx += q[0];
            sy += q[1];
            sz += q[2];
        }
        double *o = out + (long long)cl.subset * out_stride + 3ll * rperm[cl.begin + r];
        o[0] = sx;
        o[1] = sy;
        o[2] = sz;
    }
}

// The bounding box of each cluster, and for the adjoint (w != nullptr, every
// particle a receiver) the weights of its particles in sorted order.  A group
// of kFinishLanes lanes per cluster, kWave / kFinishLanes clusters per wave,
// kFinishWaves waves per block; each lane takes PPL = csize / kFinishLanes
// receivers, loaded together (the kernel is bound by the latency of the two
// dependent loads, the record and then the receivers, so fewer and fuller
// waves finish sooner), and entries past a cluster's count repeat its first
// receiver.  The cluster count is read on the device, so the launch can be
// sized by an upper bound before the count reaches the host.
template <int PPL>
__global__ __launch_bounds__(kFinishWaves * kWave) void k_cluster_finish(
    Cluster *__restrict__ clusters, const int *__restrict__ n_clusters_dev,
    const double4 *__restrict__ rp, const double *__restrict__ w, const uint8_t *__restrict__ sel,
    const int *__restrict__ perm, int fp32, double4 *__restrict__ wa) {
    constexpr int per_wave = kWave / kFinishLanes;
    const int n_clusters = *n_clusters_dev;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = blockIdx.x * kFinishWaves + (int)(threadIdx.x / kWave);
    if (wave * per_wave >= n_clusters) return;   // whole waves leave together
    const int c = wave * per_wave + lane / kFinishLanes;
    const int li = lane & (kFinishLanes - 1);
    const bool have = c < n_clusters;
    double lx = 0.0, ly = 0.0, lz = 0.0, hx = 0.0, hy = 0.0, hz = 0.0;
    if (have) {
        const int begin = clusters[c].begin, count = clusters[c].count;
        double4 x[PPL];
#pragma unroll
        for (int k = 0; k < PPL; ++k) {
            const int q = li + kFinishLanes * k;
            x[k] = rp[begin + (q < count ? q : 0)];
        }
        if (w) {
#pragma unroll
            for (int k = 0; k < PPL; ++k) {
                const int q = li + kFinishLanes * k;
                if (q >= count) continue;
                const int p = begin + q;
                double wx = 0.0, wy = 0.0, wz = 0.0;
                if (!sel || sel[p]) {   // no selector: all active
                    const double *src = w + 3 * (size_t)perm[p];
                    wx = src[0];
                    wy = src[1];
                    wz = src[2];
                }
                if (fp32)
                    reinterpret_cast<float4 *>(wa)[p] =
                        make_float4((float)wx, (float)wy, (float)wz, 0.0f);
                else
                    wa[p] = make_double4(wx, wy, wz, 0.0);
            }
        }
        lx = hx = x[0].x;
        ly = hy = x[0].y;
        lz = hz = x[0].z;
#pragma unroll
        for (int k = 1; k < PPL; ++k) {
            lx = fmin(lx, x[k].x);
            ly = fmin(ly, x[k].y);
            lz = fmin(lz, x[k].z);
            hx = fmax(hx, x[k].x);
            hy = fmax(hy, x[k].y);
            hz = fmax(hz, x[k].z);
        }
    }
    // min / max over each aligned group of kFinishLanes lanes
#pragma unroll
    for (int off = kFinishLanes >> 1; off > 0; off >>= 1) {
        lx = fmin(lx, __shfl_xor(lx, off, kWave));
        ly = fmin(ly, __shfl_xor(ly, off, kWave));
        lz = fmin(lz, __shfl_xor(lz, off, kWave));
        hx = fmax(hx, __shfl_xor(hx, off, kWave));
        hy = fmax(hy, __shfl_xor(hy, off, kWave));
        hz = fmax(hz, __shfl_xor(hz, off, kWave));
    }
    if (have && li == 0) {
        Cluster *o = clusters + c;
        o->lo[0] = lx; o->lo[1] = ly; o->lo[2] = lz;
        o->hi[0] = hx; o->hi[1] = hy; o->hi[2] = hz;
    }
}

// Several int fills in one launch, 16 bytes per store between the unaligned
// ends: region r takes the blocks from first[r] on.
__global__ void k_fill_multi(FillSet f) {
    int r = 0;
    while (r + 1 < f.count && (int)blockIdx.x >= f.first[r + 1]) ++r;
    int *__restrict__ p = f.p[r];
    const size_t n = f.n[r];
    const int v = f.v[r];
    const size_t i = (size_t)(blockIdx.x - f.first[r]) * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)(f.first[r + 1] - f.first[r]) * blockDim.x;
    const size_t mis = ((16 - ((uintptr_t)p & 15)) & 15) / sizeof(int);
    const size_t head = mis < n ? mis : n;
    const size_t n4 = (n - head) / 4;
    if (i < head) p[i] = v;
    int4 *p4 = reinterpret_cast<int4 *>(p + head);
    const int4 v4 = make_int4(v, v, v, v);
    for (size_t j = i; j < n4; j += stride) p4[j] = v4;
    if (head + 4 * n4 + i < n) p[head + 4 * n4 + i] = v;   // at most 3 ints: the first threads
}

inline unsigned grid_for(size_t n, int block) {
    size_t g = (n + block - 1) / block;
    return (unsigned)(g > 0 ? g : 1);
}

}  // namespace

hipError_t launch_cluster_finish(Cluster *clusters, const int *n_clusters_dev, size_t bound,
                                 int csize, const double4 *rp, const double *w,
                                 const uint8_t *sel, const int *perm, int fp32, double4 *wa,
                                 hipStream_t s) {
    if (bound == 0) return hipSuccess;
    const size_t per_block = (size_t)kFinishWaves * (kWave / kFinishLanes);
    if (csize != 8 && csize != 16 && csize != 32 && csize != 64) return hipErrorInvalidValue;
    auto fn = csize == 8    ? k_cluster_finish<1>
              : csize == 16 ? k_cluster_finish<2>
              : csize == 32 ? k_cluster_finish<4>
                            : k_cluster_finish<8>;
    hipLaunchKernelGGL(fn, dim3(grid_for(bound, (int)per_block)), dim3(kFinishWaves * kWave), 0,
                       s, clusters, n_clusters_dev, rp, w, sel, perm, fp32, wa);
    return hipGetLastError();
}

hipError_t launch_fill_multi(FillSet f, hipStream_t s) {
    // 16 KB per block, at most 2048 blocks per region
    for (int r = 0; r < f.count; ++r)
        f.first[r + 1] =
            f.first[r] + (f.n[r] ? (int)std::min<size_t>(grid_for(f.n[r], 4096), 2048) : 0);
    if (f.first[f.count] == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_multi, dim3((unsigned)f.first[f.count]), dim3(256), 0, s, f);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int *p, int v, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    size_t g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)g), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_fill_f64(double *p, double v, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    size_t g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)g), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

bool keys_scan_cells(size_t ncells) { return ncells <= (size_t)kKeysScan; }

hipError_t launch_keys(const double *pos, int n, const Geom &g, int *key, int *rank,
                       int *cell_count, int *done, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const size_t ncells = (size_t)g.nt3 * g.ns3;
    const int n_scan = keys_scan_cells(ncells) ? (int)ncells : 0;
    const int ppt = keys_per_thread(n);
    auto fn = ppt == 8 ? k_keys<8> : ppt == 4 ? k_keys<4> : ppt == 2 ? k_keys<2> : k_keys<1>;
    hipLaunchKernelGGL(fn, dim3(grid_for(n, kKeysThreads * ppt)), dim3(kKeysThreads), 0, s, pos, n,
                       g, key, rank, cell_count, n_scan, done);
    return hipGetLastError();
}

size_t scan_block_sums_needed(size_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

size_t scan1_status_needed(size_t n) { return n == 0 ? 1 : (n + kScanTile - 1) / kScanTile; }

hipError_t launch_scan1(const int *in, int *out, size_t n, unsigned long long *status, int *ctr,
                        unsigned long long *stall, int *bsum, hipStream_t s) {
    const size_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb == 0) {
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, out, 0, (size_t)1);
        return hipGetLastError();
    }
    // past a few dozen tiles the blocks running together wait on each
    // other's prefixes in a chain (a rung-batched flag scan of 134M values
    // took 3.9 ms with a one-lane look-back), where three launches take less
    if (nb > (size_t)kScan1MaxTiles) return launch_scan(in, out, n, bsum, s);
    hipLaunchKernelGGL(k_scan_1pass, dim3((unsigned)nb), dim3(kScanBlock), 0, s, in, out, n,
                       status, ctr, stall);
    return hipGetLastError();
}

hipError_t launch_scan(const int *in, int *out, size_t n, int *bsum, hipStream_t s) {
    size_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb == 0) {
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, out, 0, (size_t)1);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kScanBlock), 0, s, in, n, bsum);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, bsum, (int)nb, out + n);
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kScanBlock), 0, s, in, out, n, bsum);
    return hipGetLastError();
}

hipError_t launch_scatter(const double *pos, const double *mass, const uint8_t *sel, int n,
                          const Geom &g, const int *key, const int *rank, const int *cell_start,
                          int fp32, int csize, bool stable, double4 *sp, int *perm,
                          uint8_t *sel_s, double4 *sp2, int *perm2, uint8_t *sel2,
                          int *big_list, hipStream_t s) {
    if (n == 0) return hipSuccess;
    // stable ranks are already in fine order: every subtile goes straight out
    const int keep_max = stable ? INT_MAX : (csize > kFineMin ? csize : kFineMin);
    hipLaunchKernelGGL(k_scatter, dim3(grid_for(n, 256)), dim3(256), 0, s, pos, mass, sel, n, g,
                       key, rank, cell_start, fp32, keep_max, sp, perm, sel_s, sp2, perm2, sel2,
                       big_list);
    return hipGetLastError();
}

hipError_t launch_fine_order(const double4 *sp, const int *perm, const uint8_t *sel,
                             const int *cell_start, const Geom &g, int *fkey, int *frank,
                             double4 *sp2, int *perm2, uint8_t *sel2, int n, int csize,
                             const int *big_list, hipStream_t s) {
    const int big = std::min(n / kFineBig, 256);
    const long long med = std::min<long long>((g.nt3 + kFineWaves - 1) / kFineWaves, 1ll << 20);
    hipLaunchKernelGGL(k_fine_order, dim3((unsigned)(big + med)), dim3(kFineBins), 0, s, sp, perm,
                       sel, cell_start, g, fkey, frank, sp2, perm2, sel2,
                       csize > kFineMin ? csize : kFineMin, big, big_list);
    return hipGetLastError();
}

hipError_t launch_receivers(const uint8_t *sel_s, int n, int n_sub, int kind,
                            const uint8_t *thr_host, const double4 *sp, const int *perm,
                            int *prefix, double4 *rp, int *rperm, unsigned long long *status,
                            int *ctr, unsigned long long *stall, hipStream_t s) {
    const size_t rows = (size_t)n * n_sub;
    if (rows == 0) return hipSuccess;
    Thresholds thr{};
    if (thr_host)
        for (int k = 0; k < n_sub && k < 64; ++k) thr.t[k] = thr_host[k];
    hipLaunchKernelGGL(k_receivers, dim3(grid_for(rows, kRecvTile)), dim3(kRecvThreads), 0, s, sel_s,
                       n, n_sub, kind, thr, sp, perm, prefix, rp, rperm, status, ctr, stall);
    return hipGetLastError();
}

static bool plan_big(int n_sub, const Geom &g) { return (long long)n_sub * g.nt3 > kPlanBigFrom; }

size_t receivers_status_needed(size_t rows) { return (rows + kRecvTile - 1) / kRecvTile; }

size_t plan_status_needed(int n_sub, const Geom &g) {
    const size_t per = plan_big(n_sub, g) ? kPlanThreadsBig : 64;
    return ((size_t)n_sub * g.nt3 + per - 1) / per;
}

hipError_t launch_plan(const PlanArgs &p, const Geom &g, hipStream_t s) {
    const unsigned grid = (unsigned)plan_status_needed(p.n_sub, g);
    if (plan_big(p.n_sub, g))
        hipLaunchKernelGGL((p.half ? k_plan<true, kPlanThreadsBig, kPlanThreadsBig>
                                   : k_plan<false, kPlanThreadsBig, kPlanThreadsBig>),
                           dim3(grid), dim3(kPlanThreadsBig), 0, s, p, g);
    else
        hipLaunchKernelGGL((p.half ? k_plan<true, 64, kPlanThreads> : k_plan<false, 64, kPlanThreads>),
                           dim3(grid), dim3(kPlanThreads), 0, s, p, g);
    return hipGetLastError();
}

hipError_t launch_item_write(const Cluster *clusters, const int *n_clusters_dev, int bound,
                             const int *cs, const Geom &g, int target, int half, int split,
                             const int *item_off, Item *items, hipStream_t s) {
    if (bound == 0) return hipSuccess;
    hipLaunchKernelGGL(half ? k_item_write<true> : k_item_write<false>,
                       dim3(grid_for(bound, 128)), dim3(128), 0, s, clusters, n_clusters_dev, cs, g,
                       target, split, item_off, items);
    return hipGetLastError();
}

// Histogram of particles per tile in 32 bins: bin 0 empty tiles, bin b > 0
// tiles holding [2^(b-1), 2^b) particles (hist zeroed before the launch).
__global__ void k_tile_hist(const int *__restrict__ cs, Geom g, int *__restrict__ hist) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= g.nt3) return;
    const int cnt = cs[(size_t)(t + 1) * g.ns3] - cs[(size_t)t * g.ns3];
    const int b = cnt <= 0 ? 0 : min(31, 32 - __clz(cnt));
    atomicAdd(&hist[b], 1);
}

hipError_t launch_tile_hist(const int *cell_start, const Geom &g, int *hist32, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, hist32, 0, (size_t)32);
    hipLaunchKernelGGL(k_tile_hist, dim3(grid_for((size_t)g.nt3, 256)), dim3(256), 0, s,
                       cell_start, g, hist32);
    return hipGetLastError();
}

size_t stable_rank_hist_ints(int n) { return (size_t)256 * ((n + kRsTile - 1) / kRsTile); }

hipError_t launch_stable_ranks(const double *pos, int n, const Geom &g, const int *key,
                               const int *cell_start, unsigned long long *k64a,
                               unsigned long long *k64b, int *va, int *vb, int *hist, int *bsum,
                               int *rank, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const int nblk = (n + kRsTile - 1) / kRsTile;
    const long long ncells = (long long)g.nt3 * g.ns3;
    int bits = kFineBits;
    while (bits < 64 && (1ll << (bits - kFineBits)) < ncells) ++bits;
    hipLaunchKernelGGL(k_rs_keys, dim3(grid_for(n, 256)), dim3(256), 0, s, pos, n, g, key, k64a,
                       va);
    for (int shift = 0; shift < bits; shift += 8) {
        hipLaunchKernelGGL(k_rs_hist, dim3(nblk), dim3(kWave), 0, s, k64a, n, shift, nblk, hist);
        hipError_t e = launch_scan(hist, hist, (size_t)256 * nblk, bsum, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_rs_scatter, dim3(nblk), dim3(kWave), 0, s, k64a, va, n, shift, nblk,
                           hist, k64b, vb);
        std::swap(k64a, k64b);
        std::swap(va, vb);
    }
    hipLaunchKernelGGL(k_rs_rank, dim3(grid_for(n, 256)), dim3(256), 0, s, k64a, va, n,
                       cell_start, rank);
    return hipGetLastError();
}

hipError_t launch_item_reduce(const Cluster *clusters, const int *n_clusters_dev, int bound,
                              const int *item_off, const double *partials, int csize,
                              const int *rperm, double *out, long long out_stride,
                              hipStream_t s) {
    if (bound == 0) return hipSuccess;
    const int grid = std::min(bound, 65536);
    hipLaunchKernelGGL(k_item_reduce, dim3(grid), dim3(kWave), 0, s, clusters, n_clusters_dev,
                       item_off, partials, csize, rperm, out, out_stride);
    return hipGetLastError();
}

}  // namespace p3m
