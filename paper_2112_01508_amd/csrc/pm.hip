// Long-range (PM) half of the P3M gravity: CONCEPT 1.0, section 2.1.3, the
// upper half of eq. p3m_gravity, which runs the PM steps of eq. pm_method
// with the long-range kernel exp(-x_s^2 k^2) / k^2 of eq. ewald_potential:
//
//   sort       counting sort of the particles by bins of 8^3 lower CIC nodes
//   deposit    rho_m = sum_j mu_j W(x_m - x_j), CIC weights (eq. W_CIC),
//              cell-centred nodes x_m = h (m + 1/2); added in LDS brick by
//              brick, each brick stored once
//   x forward  real lines two at a time as one complex line, radix-2 FFT in
//              LDS, split into the two half spectra (kx = 0 .. n/2)
//   y forward  strided complex FFTs over tiles of adjacent kx columns
//   z          forward FFT, multiply by the kernel, inverse FFT, all in LDS
//              (one pass over HBM instead of three)
//   y inverse
//   x inverse  two half spectra rebuilt into one complex line, inverse FFT,
//              the real and imaginary parts are the two real lines of phi
//   readout    per receiver: 4-point difference (eq. symmetric_diff_4) of phi
//              at the 8 CIC nodes and CIC interpolation (eq. pm_force)
//
// The kernel applied in the z pass is
//   G(k) = 4 pi / h^4 / n^3 * exp(-x_s^2 k^2) / k^2 * prod_d sinc(h k_d / 2)^-4
// (the two CIC deconvolutions of eq. weight_fourier, the 1/n^3 of the
// normalised inverse transform and the prefactor of eq. p3m_gravity folded
// in), G(0) = 0.  It is separable apart from 1/k^2, so two tables of n
// values (per axis index: exp(-x_s^2 k_i^2) sinc^-4 and k_i^2) describe it.
//
// Layouts in HBM: real grids (rho, then phi in the same buffer) are n^3 FP64
// with x fastest, index (z n + y) n + x.  The half-spectrum grid holds
// nh = n/2 + 1 complex FP64 values per (y, z) line at a row stride rs of nh
// rounded up to 8, index (z n + y) rs + kx.
#include <hip/hip_runtime.h>

#include "p3msr_internal.hpp"

namespace p3m {
namespace {

constexpr int kFftThreads = 256;
#ifndef P3M_FFT_TILE
#define P3M_FFT_TILE 2048
#endif
constexpr int kFftTile = P3M_FFT_TILE;   // complex values per workgroup tile (16 B each)

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Wrap one coordinate into [0, box) as the oracle does (remainder, then a
// result that rounded up to box itself becomes box - box = 0).
__device__ __forceinline__ double wrap_coord(double x, double box) {
    if (x >= 0.0 && x < box) return x;   // the usual case: already in the box
    double r = fmod(x, box);
    if (r < 0.0) r += box;
    if (r >= box) r -= box;
    return r;
}

// Lower CIC node (in [0, n)) and the weight f of the upper node.
__device__ __forceinline__ int cic_node(double x, double box, double h, int n, double &f) {
    const double u = wrap_coord(x, box) / h - 0.5;
    const double i0 = floor(u);
    f = u - i0;
    return ((int)i0 + n) & (n - 1);
}

// Workgroups are dealt round-robin to the XCDs: the block's place when each
// XCD is to take a contiguous eighth of the work (gridDim.x a multiple of
// kXcds), so that neighbouring blocks' common data come from one L2.
__device__ __forceinline__ int xcd_block() {
    return (int)(blockIdx.x % kXcds) * (int)(gridDim.x / kXcds) + (int)(blockIdx.x / kXcds);
}

// Counting sort of the particles by bins of 8^3 lower CIC nodes (index (bz nb
// + by) nb + bx): rank inside the bin, then a scatter to start[bin] + rank.
// The sorted record holds the CIC fractions and mu, so the deposit and the
// readout need neither the positions nor a division.  A bin's particles are
// about one wave at mean density, and the phi values around it (13^3, 17 KB)
// fit the L1, which is all the order that deposit and readout use; a sort by
// single nodes needed a counter per node (for 2^21 particles on 256^3 nodes: an
// atomic per particle on 67 MB of counters, clearing and scanning them, 0.26 ms
// together; by bins, keys, scan and scatter take 0.11 ms).
template <int PPT>
__global__ __launch_bounds__(kKeysThreads) void k_pm_keys(const double *__restrict__ pos,
                                                          int n_part, int n, double box, double h,
                                                          int *__restrict__ key,
                                                          int *__restrict__ rank,
                                                          int *__restrict__ count) {
    const int nb = n / kPmBin;
    block_ranks<PPT>(n_part, key, rank, count, [&](size_t i) {
        double f;
        const int bx = cic_node(pos[3 * i], box, h, n, f) / kPmBin;
        const int by = cic_node(pos[3 * i + 1], box, h, n, f) / kPmBin;
        const int bz = cic_node(pos[3 * i + 2], box, h, n, f) / kPmBin;
        return (bz * nb + by) * nb + bx;
    });
}

// The deposit's blocks take the first kOverRun particles of a bin; the runs of
// kOverRun after them are listed here.
constexpr int kOverRun = 2048;

// (Writing only the sorted index here and building the records in sorted
// order with gathered reads took as long.)
__global__ void k_pm_scatter(const double *__restrict__ pos, const double *__restrict__ mass,
                             const uint8_t *__restrict__ active, int n_part, int n, double box,
                             double h, const int *__restrict__ key, const int *__restrict__ rank,
                             const int *__restrict__ start, int *__restrict__ over,
                             double4 *__restrict__ rec, int *__restrict__ nkey,
                             int *__restrict__ perm) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_part) return;
    const int k = key[i], q = rank[i];
    const int dst = start[k] + q;
    if (q >= kOverRun && q % kOverRun == 0) {
        const int at = atomicAdd(over, 1);
        over[1 + 2 * at] = k;
        over[2 + 2 * at] = dst;
    }
    double4 r;
    const int ix = cic_node(pos[3 * (size_t)i], box, h, n, r.x);
    const int iy = cic_node(pos[3 * (size_t)i + 1], box, h, n, r.y);
    const int iz = cic_node(pos[3 * (size_t)i + 2], box, h, n, r.z);
    r.w = mass ? mass[i] : 1.0;
    rec[dst] = r;
    nkey[dst] = (iz * n + iy) * n + ix;
    perm[dst] = active && !active[i] ? ~i : i;
}

// CIC deposit.  One block owns B^3 grid nodes (B = 16, or 8 on a 16^3 grid)
// and takes the particles of the bins that reach them: its own and the next
// lower ones, (B / 8 + 1)^3 in all.  Each adds those of its 8 weights that
// fall into the brick in LDS, and the brick is stored, so this needs neither
// global atomics nor a cleared grid.  Every bin is read by up to 8 bricks
// (3.4 on average); the reads come from the caches.  2^21 clustered particles
// on 256^3 nodes: 0.089 ms, and 0.009 for the runs of dense bins below (0.117
// and 0.015 when single nodes were sorted and looked up here).
template <int kBrick>
__global__ __launch_bounds__(512) void k_pm_deposit_brick(const double4 *__restrict__ rec,
                                                          const int *__restrict__ nkey,
                                                          const int *__restrict__ start, int n,
                                                          int lg, double *__restrict__ rho) {
    constexpr int kThreads = 512;
    constexpr int kSide = kBrick / kPmBin + 1;
    constexpr int kBins = kSide * kSide * kSide;
    __shared__ double acc[kBrick * kBrick * kBrick];
    __shared__ int first[kBins], pre[kBins + 1];
    const int t = threadIdx.x;
    const int msk = n - 1, nb8 = n / kPmBin;
    const int nb = n / kBrick;
    const int b = xcd_block();
    const int x0 = (b % nb) * kBrick, y0 = ((b / nb) % nb) * kBrick, z0 = (b / (nb * nb)) * kBrick;
    for (int j = t; j < kBrick * kBrick * kBrick; j += kThreads) acc[j] = 0.0;
    if (t < kWave) {
        int len = 0;
        if (t < kBins) {
            const int bx = (x0 / kPmBin - 1 + t % kSide) & (nb8 - 1);
            const int by = (y0 / kPmBin - 1 + (t / kSide) % kSide) & (nb8 - 1);
            const int bz = (z0 / kPmBin - 1 + t / (kSide * kSide)) & (nb8 - 1);
            const int c = (bz * nb8 + by) * nb8 + bx;
            first[t] = start[c];
            len = min(start[c + 1] - start[c], kOverRun);
        }
        int incl = len;
        for (int off = 1; off < kWave; off <<= 1) {
            const int y = __shfl_up(incl, off, kWave);
            if (t >= off) incl += y;
        }
        if (t < kBins) pre[t + 1] = incl;
        if (t == 0) pre[0] = 0;
    }
    __syncthreads();
    const int total = pre[kBins];
    for (int i = t; i < total; i += kThreads) {
        // the bin holding entry i: the last j with pre[j] <= i
        int lo = 0, hi = kBins;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= i) lo = mid;
            else hi = mid;
        }
        const int q = first[lo] + (i - pre[lo]);
        const int k = nkey[q];
        const double4 r = rec[q];   // loaded beside the key, not after it
        // the lower node relative to the brick, -1 .. kBrick - 1 where it reaches it
        const int x = (((k & msk) - x0 + 1) & msk) - 1;
        const int y = ((((k >> lg) & msk) - y0 + 1) & msk) - 1;
        const int z = (((k >> (2 * lg)) - z0 + 1) & msk) - 1;
        if (x >= kBrick || y >= kBrick || z >= kBrick) continue;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int tx = x + ((c >> 2) & 1), ty = y + ((c >> 1) & 1), tz = z + (c & 1);
            if ((unsigned)tx < kBrick && (unsigned)ty < kBrick && (unsigned)tz < kBrick) {
                const double wx = (c & 4) ? r.x : 1.0 - r.x;
                const double wy = (c & 2) ? r.y : 1.0 - r.y;
                const double wz = (c & 1) ? r.z : 1.0 - r.z;
                atomicAdd(&acc[(tz * kBrick + ty) * kBrick + tx], r.w * wx * wy * wz);
            }
        }
    }
    __syncthreads();
    for (int j = t; j < kBrick * kBrick * kBrick; j += kThreads) {
        const int tx = j % kBrick, ty = (j / kBrick) % kBrick, tz = j / (kBrick * kBrick);
        rho[((size_t)(z0 + tz) * n + (y0 + ty)) * n + (x0 + tx)] = acc[j];
    }
}

// The listed runs of dense bins, one block each: their weights are added in
// LDS on the (8 + 1)^3 nodes that a bin reaches, and those sums on top of the
// bricks with one global atomic per node.
__global__ __launch_bounds__(256) void k_pm_deposit_over(const double4 *__restrict__ rec,
                                                         const int *__restrict__ nkey,
                                                         const int *__restrict__ start,
                                                         const int *__restrict__ over, int n,
                                                         int lg, double *__restrict__ rho) {
    constexpr int S = kPmBin + 1;
    __shared__ double acc[S * S * S];
    const int msk = n - 1, nb = n / kPmBin;
    const int runs = over[0];
    for (int e = blockIdx.x; e < runs; e += gridDim.x) {
        const int bin = over[1 + 2 * e], q0 = over[2 + 2 * e];
        const int q1 = min(q0 + kOverRun, start[bin + 1]);
        const int x0 = (bin % nb) * kPmBin, y0 = ((bin / nb) % nb) * kPmBin,
                  z0 = (bin / (nb * nb)) * kPmBin;
        for (int j = threadIdx.x; j < S * S * S; j += blockDim.x) acc[j] = 0.0;
        __syncthreads();
        for (int q = q0 + threadIdx.x; q < q1; q += blockDim.x) {
            const int k = nkey[q];
            const int x = (k & msk) - x0, y = ((k >> lg) & msk) - y0, z = (k >> (2 * lg)) - z0;
            const double4 r = rec[q];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const double wx = (c & 4) ? r.x : 1.0 - r.x;
                const double wy = (c & 2) ? r.y : 1.0 - r.y;
                const double wz = (c & 1) ? r.z : 1.0 - r.z;
                atomicAdd(&acc[((z + (c & 1)) * S + y + ((c >> 1) & 1)) * S + x + ((c >> 2) & 1)],
                          r.w * wx * wy * wz);
            }
        }
        __syncthreads();
        for (int j = threadIdx.x; j < S * S * S; j += blockDim.x) {
            const size_t x = (x0 + j % S) & msk, y = (y0 + (j / S) % S) & msk,
                         z = (z0 + j / (S * S)) & msk;
            if (acc[j] != 0.0) atomicAdd(rho + (z * n + y) * n + x, acc[j]);
        }
        __syncthreads();
    }
}

// Twiddles tw[m] = exp(-2 pi i m / n), m < n/2, the kernel tables, and the
// sort array (16-byte stores; its length is a multiple of 4 ints) and *stall
// cleared.
__global__ void k_pm_prepare(int n, double box, double x_s, double2 *tw, double *w1, double *k2,
                             int4 *zero, size_t n4, unsigned long long *stall) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *stall = 0;
    for (size_t j = i; j < n4; j += (size_t)gridDim.x * blockDim.x) zero[j] = make_int4(0, 0, 0, 0);
    if (i < n / 2) {
        double s, c;
        sincospi(2.0 * (double)i / (double)n, &s, &c);
        tw[i] = make_double2(c, -s);
    }
    if (i < n) {
        const int hh = i < n / 2 ? i : i - n;
        const double k = 2.0 * M_PI * (double)hh / box;
        double sinc = 1.0;
        if (hh != 0) {
            const double t = (double)hh / (double)n;
            sinc = sinpi(t) / (M_PI * t);
        }
        const double s2 = sinc * sinc;
        k2[i] = k * k;
        w1[i] = exp(-x_s * x_s * k * k) / (s2 * s2);
    }
}

// Copies the n/2 twiddles into LDS (the caller synchronises before use).
template <int N>
__device__ __forceinline__ void stage_twiddles(double2 *tws, const double2 *__restrict__ tw) {
    for (int k = threadIdx.x; k < N / 2; k += kFftThreads) tws[k] = tw[k];
}

// Twiddle exp(-2 pi i m / N) for 0 <= m < N from the half table tw[m < N/2].
template <int N>
__device__ __forceinline__ double2 twiddle(const double2 *tw, int m) {
    if (m < N / 2) return tw[m];
    const double2 w = tw[m - N / 2];
    return make_double2(-w.x, -w.y);
}

// One radix-R Stockham stage (R = 2 or 4) at span Ns: butterfly j reads
// x_q = x[j + q N/R], multiplies x_q by w^(q k) with w = exp(-+2 pi i /
// (R Ns)) and k = j mod Ns, takes the R-point DFT and writes output q to
// (j - k) R + k + q Ns.
template <int N, int LINES, int IS, int LS, bool LANE_J, bool INV, int R>
__device__ __forceinline__ void fft_stage(double2 *buf, const double2 *tw, int Ns) {
    constexpr int NB = LINES * (N / R);
    constexpr int PER = (NB + kFftThreads - 1) / kFftThreads;
    const int t = threadIdx.x;
    const int step = N / (R * Ns);   // twiddle table stride per unit of q k
    double2 y[PER][R];
    int dst[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int bi = t + u * kFftThreads;
        if (NB % kFftThreads == 0 || bi < NB) {
            const int j = LANE_J ? bi % (N / R) : bi / LINES;
            const int l = LANE_J ? bi / (N / R) : bi % LINES;
            const int k = j & (Ns - 1);
            double2 x[R];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                x[q] = buf[(j + q * (N / R)) * IS + l * LS];
                if (q > 0) {
                    double2 w = twiddle<N>(tw, q * k * step);
                    if (INV) w.y = -w.y;
                    x[q] = cmul(x[q], w);
                }
            }
            if constexpr (R == 2) {
                y[u][0] = make_double2(x[0].x + x[1].x, x[0].y + x[1].y);
                y[u][1] = make_double2(x[0].x - x[1].x, x[0].y - x[1].y);
            } else {
                const double2 a0 = make_double2(x[0].x + x[2].x, x[0].y + x[2].y);
                const double2 a1 = make_double2(x[0].x - x[2].x, x[0].y - x[2].y);
                const double2 a2 = make_double2(x[1].x + x[3].x, x[1].y + x[3].y);
                const double2 d = make_double2(x[1].x - x[3].x, x[1].y - x[3].y);
                // a3 = d * (-i) forward, d * (+i) inverse
                const double2 a3 = INV ? make_double2(-d.y, d.x) : make_double2(d.y, -d.x);
                y[u][0] = make_double2(a0.x + a2.x, a0.y + a2.y);
                y[u][1] = make_double2(a1.x + a3.x, a1.y + a3.y);
                y[u][2] = make_double2(a0.x - a2.x, a0.y - a2.y);
                y[u][3] = make_double2(a1.x - a3.x, a1.y - a3.y);
            }
            dst[u] = ((j - k) * R + k) * IS + l * LS;
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int bi = t + u * kFftThreads;
        if (NB % kFftThreads == 0 || bi < NB) {
#pragma unroll
            for (int q = 0; q < R; ++q) buf[dst[u] + q * Ns * IS] = y[u][q];
        }
    }
    __syncthreads();
}

// FFT of `lines` lines of length N held in LDS.  Element (l, i) sits at
// i * IS + l * LS.  Mixed-radix Stockham: radix-4 stages, after one radix-2
// stage when log2 N is odd; the result comes out in natural order without a
// bit reversal.  lane_j: consecutive threads take consecutive j (line-major
// tiles) or consecutive lines (interleaved tiles).
template <int N, int LINES, int IS, int LS, bool LANE_J, bool INV>
__device__ __forceinline__ void lds_fft(double2 *buf, const double2 *tw) {
    constexpr int LOG = __builtin_ctz(N);
    int Ns = 1;
    if constexpr (LOG % 2 == 1) {
        fft_stage<N, LINES, IS, LS, LANE_J, INV, 2>(buf, tw, 1);
        Ns = 2;
    }
#pragma unroll 1
    for (; Ns < N; Ns *= 4) fft_stage<N, LINES, IS, LS, LANE_J, INV, 4>(buf, tw, Ns);
}

// Half-spectrum rows hold NH = N/2 + 1 values, stored with a stride rounded
// up to 8 complex values (128 B) so that column tiles start on cache lines.
template <int N>
struct Row {
    static constexpr int kNH = N / 2 + 1;
    static constexpr int kStride = (kNH + 7) & ~7;
};

template <int N>
struct XTile {
    static constexpr int kLines = (kFftTile / N) < (N * N / 2) ? (kFftTile / N) : (N * N / 2);
};

// x forward: real lines 2p, 2p+1 of rho as the real and imaginary parts of
// one complex line; after the FFT Z, A_k = (Z_k + conj Z_{N-k}) / 2 and
// B_k = -i (Z_k - conj Z_{N-k}) / 2 are the spectra of the two real lines.
template <int N>
__global__ __launch_bounds__(kFftThreads) void k_fft_x_fwd(const double *__restrict__ rho,
                                                           double2 *__restrict__ spec,
                                                           const double2 *__restrict__ tw) {
    constexpr int P = XTile<N>::kLines;     // complex lines per tile
    constexpr int NH = N / 2 + 1;
    __shared__ double2 buf[P * N];
    __shared__ double2 tws[N / 2];
    stage_twiddles<N>(tws, tw);
    const size_t line0 = (size_t)blockIdx.x * 2 * P;   // first real line of the tile
    const double *src = rho + line0 * N;
    double *bufd = reinterpret_cast<double *>(buf);
    for (int e = threadIdx.x; e < 2 * P * N; e += kFftThreads) {
        const int r = e / N, i = e % N;
        bufd[2 * ((r >> 1) * N + i) + (r & 1)] = src[e];
    }
    __syncthreads();
    lds_fft<N, P, 1, N, true, false>(buf, tws);
    double2 *dst = spec + line0 * Row<N>::kStride;
    // both half spectra of a line pair from one read of Z_k and Z_{N-k}
    for (int e = threadIdx.x; e < P * NH; e += kFftThreads) {
        const int p = e / NH, k = e % NH;
        const double2 z = buf[p * N + k];
        const double2 zc = buf[p * N + ((N - k) & (N - 1))];   // enters conjugated
        dst[(size_t)(2 * p) * Row<N>::kStride + k] =
            make_double2(0.5 * (z.x + zc.x), 0.5 * (z.y - zc.y));
        dst[(size_t)(2 * p + 1) * Row<N>::kStride + k] =
            make_double2(0.5 * (z.y + zc.y), -0.5 * (z.x - zc.x));
    }
}

// x inverse: Z_k = A_k + i B_k (k <= N/2), conj(A_{N-k}) + i conj(B_{N-k})
// above; the inverse FFT of Z holds line 2p in its real part and line 2p+1
// in its imaginary part.
template <int N>
__global__ __launch_bounds__(kFftThreads) void k_fft_x_inv(const double2 *__restrict__ spec,
                                                           double *__restrict__ phi,
                                                           const double2 *__restrict__ tw) {
    constexpr int P = XTile<N>::kLines;
    constexpr int NH = N / 2 + 1;
    __shared__ double2 buf[P * N];
    __shared__ double2 tws[N / 2];
    stage_twiddles<N>(tws, tw);
    const size_t line0 = (size_t)blockIdx.x * 2 * P;
    const double2 *src = spec + line0 * Row<N>::kStride;
    for (int e = threadIdx.x; e < P * N; e += kFftThreads) {
        const int p = e / N, k = e % N;
        const bool lo = k <= N / 2;
        const int kk = lo ? k : N - k;
        const double2 a = src[(size_t)(2 * p) * Row<N>::kStride + kk];
        const double2 b = src[(size_t)(2 * p + 1) * Row<N>::kStride + kk];
        buf[e] = lo ? make_double2(a.x - b.y, a.y + b.x) : make_double2(a.x + b.y, b.x - a.y);
    }
    __syncthreads();
    lds_fft<N, P, 1, N, true, true>(buf, tws);
    double *dst = phi + line0 * N;
    const double *bufd = reinterpret_cast<const double *>(buf);
    for (int e = threadIdx.x; e < 2 * P * N; e += kFftThreads) {
        const int r = e / N, i = e % N;
        dst[e] = bufd[2 * ((r >> 1) * N + i) + (r & 1)];
    }
}

template <int N>
struct STile {
    // 4..16 adjacent columns: rows are read at least 64 B at a time
    static constexpr int kRaw = kFftTile / N;
    static constexpr int kCols = kRaw < 4 ? 4 : (kRaw > 16 ? 16 : kRaw);
};

// Strided passes over tiles of C adjacent kx columns.  AXIS 1 (y): blockIdx.y
// is z, elements step by the row stride.  AXIS 2 (z): blockIdx.y is y,
// elements step by N row strides.  CONV: forward FFT, multiply by the kernel,
// inverse FFT.
template <int N, int AXIS, int MODE>   // MODE 0 forward, 1 inverse, 2 convolve
__global__ __launch_bounds__(kFftThreads) void k_fft_strided(double2 *__restrict__ spec,
                                                             const double2 *__restrict__ tw,
                                                             const double *__restrict__ w1,
                                                             const double *__restrict__ k2,
                                                             double scale) {
    constexpr int C = STile<N>::kCols;
    constexpr int NH = N / 2 + 1;
    __shared__ double2 buf[C * N];
    __shared__ double2 tws[N / 2];
    stage_twiddles<N>(tws, tw);
    const int kx0 = blockIdx.x * C;
    const int other = blockIdx.y;   // z for the y pass, y for the z pass
    constexpr size_t RS = Row<N>::kStride;
    const size_t base = AXIS == 1 ? (size_t)other * N * RS + kx0 : (size_t)other * RS + kx0;
    const size_t step = AXIS == 1 ? RS : (size_t)N * RS;
    const int ncol = NH - kx0 < C ? NH - kx0 : C;
    for (int e = threadIdx.x; e < C * N; e += kFftThreads) {
        const int c = e % C, i = e / C;
        buf[e] = c < ncol ? spec[base + (size_t)i * step + c] : make_double2(0.0, 0.0);
    }
    __syncthreads();
    if (MODE == 1) {
        lds_fft<N, C, C, 1, false, true>(buf, tws);
    } else {
        lds_fft<N, C, C, 1, false, false>(buf, tws);
    }
    if (MODE == 2) {
        // element (c, kz) of column kx = kx0 + c on the line ky = other
        const double wy = w1[other], ky2 = k2[other];
        for (int e = threadIdx.x; e < C * N; e += kFftThreads) {
            const int c = e % C, kz = e / C;
            const int kx = kx0 + c;
            if (c < ncol) {
                const double kk = k2[kx] + ky2 + k2[kz];
                const double g = kk > 0.0 ? scale * (w1[kx] * wy * w1[kz]) / kk : 0.0;
                buf[e] = make_double2(buf[e].x * g, buf[e].y * g);
            }
        }
        __syncthreads();
        lds_fft<N, C, C, 1, false, true>(buf, tws);
    }
    for (int e = threadIdx.x; e < C * N; e += kFftThreads) {
        const int c = e % C, i = e / C;
        if (c < ncol) spec[base + (size_t)i * step + c] = buf[e];
    }
}

// Readout: per receiver, the 4-point difference of phi along each axis at the
// 8 CIC nodes and their CIC-weighted sum.  The stencil is the four x rows of
// the node pairs in y and z (six values each: D4 at both x nodes), and for the
// differences along y and z the two x nodes of the 16 rows at distance 1 and 2
// from them, interpolated along x first: 28 pairs of x neighbours.
//
// The kernel is bound by its gathers: each lane's row is a cache line of its
// own, and the address unit takes a lane per cycle whatever the load's width
// (64 accesses per load and wave by its counters).  So the pairs are loaded 16
// bytes at a time, 28 loads instead of 72: 2^21 particles on 256^3 nodes 0.219
// -> 0.182 ms, 262144 on 128^3 0.031 -> 0.022 ms, although the particles are no
// longer sorted by node, which let some of the 72 share lines.  (Staging phi
// per 16^3-node brick in LDS and reading the stencils from there took 0.222 ms,
// 0.106 of it for the staging alone.)
__device__ __forceinline__ double d4_of(double a, double b, double c, double d) {
    return (a - 8.0 * b + 8.0 * c - d) / 12.0;   // phi[m-2], [m-1], [m+1], [m+2]
}

// Two values on any 8-byte boundary, as one 16-byte load.
typedef double Pair8 __attribute__((ext_vector_type(2), aligned(8)));

__global__ __launch_bounds__(256) void k_pm_readout(const double4 *__restrict__ rec,
                                                    const int *__restrict__ nkey,
                                                    const int *__restrict__ perm, int n_part,
                                                    const double *__restrict__ phi, int n, int lg,
                                                    double *__restrict__ acc) {
    const long long at = (long long)xcd_block() * blockDim.x + threadIdx.x;
    if (at >= n_part) return;
    const int p = (int)at;
    const int who = perm[p];
    double ox = 0.0, oy = 0.0, oz = 0.0;
    if (who >= 0) {
        const double4 r = rec[p];
        const int key = nkey[p];
        const int m = n - 1;
        const int ix = key & m, iy = (key >> lg) & m, iz = key >> (2 * lg);
        // values x, x + 1 of a row (x already wrapped): the pair past the
        // row's end wraps to its start
        auto pair = [&](const double *row, int x) {
            if (x == m) return make_double2(row[m], row[0]);
            const Pair8 v = *reinterpret_cast<const Pair8 *>(row + x);
            return make_double2(v.x, v.y);
        };
        const double gx = 1.0 - r.x, gy = 1.0 - r.y, gz = 1.0 - r.z;
        const int xm = (ix - 2) & m, xp = (ix + 2) & m;
        size_t ry[6], rz[6];
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            ry[s] = (size_t)((iy - 2 + s) & m) * n;
            rz[s] = (size_t)((iz - 2 + s) & m) * n * n;
        }
        double c[2][2];   // x-interpolated values of the central rows
#pragma unroll
        for (int a = 0; a < 2; ++a) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const double *row = phi + ry[2 + a] + rz[2 + b];
                const double2 l = pair(row, xm), q = pair(row, ix), h = pair(row, xp);
                const double line = gx * d4_of(l.x, l.y, q.y, h.x) + r.x * d4_of(l.y, q.x, h.x, h.y);
                ox += (a ? r.y : gy) * (b ? r.z : gz) * line;
                c[a][b] = gx * q.x + r.x * q.y;
            }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            double y[4], z[4];   // rows -2, -1, +2, +3 along y (at node b of z), along z (at b of y)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int o = s < 2 ? s : s + 2;
                const double2 u = pair(phi + ry[o] + rz[2 + b], ix);
                const double2 v = pair(phi + ry[2 + b] + rz[o], ix);
                y[s] = gx * u.x + r.x * u.y;
                z[s] = gx * v.x + r.x * v.y;
            }
            oy += (b ? r.z : gz) * (gy * d4_of(y[0], y[1], c[1][b], y[2]) +
                                    r.y * d4_of(y[1], c[0][b], y[2], y[3]));
            oz += (b ? r.y : gy) * (gz * d4_of(z[0], z[1], c[b][1], z[2]) +
                                    r.z * d4_of(z[1], c[b][0], z[2], z[3]));
        }
    }
    // who < 0: ~particle, which receives nothing
    const size_t i = (size_t)(who >= 0 ? who : ~who);
    acc[3 * i] = ox;
    acc[3 * i + 1] = oy;
    acc[3 * i + 2] = oz;
}

template <int N>
hipError_t launch_fft_chain_n(const PmArgs &a, hipStream_t s, hipEvent_t *ev) {
    constexpr int NH = N / 2 + 1;
    constexpr int P = XTile<N>::kLines;
    constexpr int C = STile<N>::kCols;
    const int x_blocks = (N * N) / (2 * P);
    const dim3 s_grid((NH + C - 1) / C, N);
    hipError_t e;
    k_fft_x_fwd<N><<<x_blocks, kFftThreads, 0, s>>>(a.real, a.spec, a.tw);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[0], s)) != hipSuccess) return e;
    k_fft_strided<N, 1, 0><<<s_grid, kFftThreads, 0, s>>>(a.spec, a.tw, a.w1, a.k2, a.scale);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[1], s)) != hipSuccess) return e;
    k_fft_strided<N, 2, 2><<<s_grid, kFftThreads, 0, s>>>(a.spec, a.tw, a.w1, a.k2, a.scale);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[2], s)) != hipSuccess) return e;
    k_fft_strided<N, 1, 1><<<s_grid, kFftThreads, 0, s>>>(a.spec, a.tw, a.w1, a.k2, a.scale);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[3], s)) != hipSuccess) return e;
    k_fft_x_inv<N><<<x_blocks, kFftThreads, 0, s>>>(a.spec, a.real, a.tw);
    return hipGetLastError();
}

}  // namespace

PmSort pm_sort_layout(int *bins, int n, int n_part) {
    const size_t nb = (size_t)n / kPmBin, cells = nb * nb * nb;
    auto even = [](size_t v) { return (v + 3) & ~(size_t)3; };
    PmSort p{};
    size_t at = 0;
    p.start = bins;
    at += even(cells + 1);
    p.over = bins + at;
    at += even(1 + 2 * ((size_t)n_part / kOverRun + 1));
    p.status = (unsigned long long *)(bins + at);
    at += even(2 * scan1_status_needed(cells));
    p.ctr = bins + at;
    p.ints = at + 4;
    return p;
}

hipError_t launch_pm_prepare(int n, double box, double x_s, double2 *tw, double *w1, double *k2,
                             const PmSort &ps, hipStream_t s) {
    const size_t n4 = ps.ints / 4;
    const size_t blocks = (n4 + 1023) / 1024;
    const unsigned grid = (unsigned)(blocks < (size_t)n / 256 + 1 ? n / 256 + 1
                                     : blocks > 4096              ? 4096
                                                                  : blocks);
    k_pm_prepare<<<grid, 256, 0, s>>>(n, box, x_s, tw, w1, k2, (int4 *)ps.start, n4, ps.stall);
    return hipGetLastError();
}

hipError_t launch_pm_sort(const double *pos, const double *mass, const uint8_t *active,
                          int n_part, int n, double box, double h, int *key, int *rank,
                          const PmSort &ps, int *bsum, double4 *rec, int *nkey, int *perm,
                          hipStream_t s) {
    if (n_part == 0) return hipSuccess;
    const size_t nb = (size_t)n / kPmBin, cells = nb * nb * nb;
    const int ppt = keys_per_thread(n_part);
    auto fn = ppt == 8   ? k_pm_keys<8>
              : ppt == 4 ? k_pm_keys<4>
              : ppt == 2 ? k_pm_keys<2>
                         : k_pm_keys<1>;
    const int per = kKeysThreads * ppt;
    fn<<<(unsigned)((n_part + per - 1) / per), kKeysThreads, 0, s>>>(pos, n_part, n, box, h, key,
                                                                     rank, ps.start);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // start[k] = first sorted index of bin k
    if ((e = launch_scan1(ps.start, ps.start, cells, ps.status, ps.ctr, ps.stall, bsum, s)) !=
        hipSuccess)
        return e;
    k_pm_scatter<<<(unsigned)((n_part + 255) / 256), 256, 0, s>>>(
        pos, mass, active, n_part, n, box, h, key, rank, ps.start, ps.over, rec, nkey, perm);
    return hipGetLastError();
}

hipError_t launch_pm_deposit(const double4 *rec, const int *nkey, const PmSort &ps, int n_part,
                             double *rho, int n, hipStream_t s) {
    const int lg = __builtin_ctz((unsigned)n);
    if (n >= 32) {
        const unsigned nb = (unsigned)n / 16;
        k_pm_deposit_brick<16><<<nb * nb * nb, 512, 0, s>>>(rec, nkey, ps.start, n, lg, rho);
    } else {
        const unsigned nb = (unsigned)n / 8;
        k_pm_deposit_brick<8><<<nb * nb * nb, 512, 0, s>>>(rec, nkey, ps.start, n, lg, rho);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_part <= kOverRun) return e;
    const int runs = n_part / kOverRun;
    k_pm_deposit_over<<<(unsigned)(runs < 1024 ? runs : 1024), 256, 0, s>>>(rec, nkey, ps.start,
                                                                          ps.over, n, lg, rho);
    return hipGetLastError();
}

hipError_t launch_pm_fft_chain(const PmArgs &a, hipStream_t s, hipEvent_t *ev) {
    switch (a.n) {
        case 16: return launch_fft_chain_n<16>(a, s, ev);
        case 32: return launch_fft_chain_n<32>(a, s, ev);
        case 64: return launch_fft_chain_n<64>(a, s, ev);
        case 128: return launch_fft_chain_n<128>(a, s, ev);
        case 256: return launch_fft_chain_n<256>(a, s, ev);
        case 512: return launch_fft_chain_n<512>(a, s, ev);
        case 1024: return launch_fft_chain_n<1024>(a, s, ev);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_pm_readout(const double4 *rec, const int *nkey, const int *perm, int n_part,
                             const double *phi, int n, double *acc, hipStream_t s) {
    if (n_part == 0) return hipSuccess;
    const unsigned per_xcd = (unsigned)((n_part + 256 * kXcds - 1) / (256 * kXcds));
    k_pm_readout<<<per_xcd * kXcds, 256, 0, s>>>(rec, nkey, perm, n_part, phi, n,
                                                 __builtin_ctz((unsigned)n), acc);
    return hipGetLastError();
}

}  // namespace p3m
