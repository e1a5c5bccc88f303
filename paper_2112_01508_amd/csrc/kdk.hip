// Rung-hierarchical kick-drift-kick step (CONCEPT 1.0, section 2.2.2,
// "Individual time steps", the time-stepping figure and eq. rung) in a
// static box: drift x += v tau, kick v += a dt_kick.
//
// Time is counted in integer units of tau / 2, tau = dt / 2^L the drift
// sub-step (L the highest rung of the period).  Rung l kicks every
// span(l) = 2^(L+1-l) units.  Each particle carries the time of its
// momentum (t_q) and of its next kick (t_next); a kick at time t brings the
// momentum to t + span(rung) / 2, or to the period's end at the last kick.
// The host loop (api.hip) evaluates the short-range force with the particles
// due at t as receivers and calls k_kdk_advance, which kicks them, drifts
// everyone over tau and marks and counts the particles due at t + 2; where the
// long-range force kicks everyone (whenever rung 0 kicks), between the short
// kick and the drift, those two are calls of their own.
#include <hip/hip_runtime.h>

#include "p3msr_internal.hpp"

namespace p3m {
namespace {

// eq. rung: max(0, ceil(log2(dt sqrt(|a| / (2 eta eps))))), capped.  The
// ceiling of log2 is read off the binary exponent, exactly.
__device__ __forceinline__ int rung_of(double ax, double ay, double az, const KdkArgs &k) {
    const double mag = sqrt(__dadd_rn(__dadd_rn(__dmul_rn(ax, ax), __dmul_rn(ay, ay)),
                                      __dmul_rn(az, az)));
    if (!(mag > 0.0)) return 0;
    const double z = k.dt * sqrt(mag / k.two_eta_eps);
    int e;
    const double m = frexp(z, &e);   // z = m 2^e, m in [0.5, 1)
    int l = m == 0.5 ? e - 1 : e;
    l = l < 0 ? 0 : l;
    return l > k.max_rung ? k.max_rung : l;
}

__device__ __forceinline__ int span_of(int l, int L) { return 1 << (L + 1 - l); }

// census: [0 .. 7] particles per rung, [8] the highest rung.  Counted per
// block first: one device atomic per particle on the same address took 25 us
// for 110592 particles.
__global__ void k_kdk_assign(const double *__restrict__ acc, int n, KdkArgs k,
                             uint8_t *__restrict__ rung, int *__restrict__ census) {
    __shared__ int cnt[9];
    if (threadIdx.x < 9) cnt[threadIdx.x] = 0;
    __syncthreads();
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        int l;
        if (k.fixed) {
            l = rung[i];
        } else {
            l = rung_of(acc[3 * (size_t)i], acc[3 * (size_t)i + 1], acc[3 * (size_t)i + 2], k);
            rung[i] = (uint8_t)l;
        }
        if (l < 8) atomicAdd(&cnt[l], 1);
        atomicMax(&cnt[8], l);
    }
    __syncthreads();
    if (threadIdx.x < 8 && cnt[threadIdx.x]) atomicAdd(&census[threadIdx.x], cnt[threadIdx.x]);
    if (threadIdx.x == 8) atomicMax(&census[8], cnt[8]);
}

// The half kicks from the synchronised start.
__global__ void k_kdk_first(double *__restrict__ vel, const double *__restrict__ acc, int n,
                            KdkArgs k, const uint8_t *__restrict__ rung, int *__restrict__ t_q,
                            int *__restrict__ t_next) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int sp = span_of(rung[i], k.L);
    const int target = sp / 2;
    const double dk = (double)target * k.half_tau;
    for (int d = 0; d < 3; ++d) vel[3 * (size_t)i + d] = vel[3 * (size_t)i + d] + acc[3 * (size_t)i + d] * dk;
    t_q[i] = target;
    t_next[i] = sp;
}

// The kick of a due particle at time t (v += a dk) and its rung's update.
__device__ __forceinline__ void kick(double (&v)[3], const double *__restrict__ a, int i, int t,
                                     const KdkArgs &k, uint8_t *__restrict__ rung,
                                     int *__restrict__ t_q, int *__restrict__ t_next) {
    const double ax = a[3 * (size_t)i], ay = a[3 * (size_t)i + 1], az = a[3 * (size_t)i + 2];
    int l = rung[i];
    const bool last = t == k.period;
    const int target = last ? k.period : t + span_of(l, k.L) / 2;
    const double dk = (double)(target - t_q[i]) * k.half_tau;
    v[0] = v[0] + ax * dk;
    v[1] = v[1] + ay * dk;
    v[2] = v[2] + az * dk;
    t_q[i] = target;
    if (k.fixed) {
        if (!last) t_next[i] = t + span_of(l, k.L);
        return;
    }
    const int want = rung_of(ax, ay, az, k);
    if (last) {
        rung[i] = (uint8_t)want;   // the next period's rung (uncapped by L)
        return;
    }
    const int w = want < k.L ? want : k.L;
    if (w > l) {
        l = l + 1;
    } else if (w < l && (t + span_of(l, k.L)) % span_of(l - 1, k.L) == 0) {
        l = l - 1;
    }
    rung[i] = (uint8_t)l;
    const int sp = span_of(l, k.L);
    t_next[i] = (t / sp + 1) * sp;
}

// What happens to a particle between two force calls: its kick at time t if it
// is due (KICK), then the drift over tau and whether it is due at t + 2 (DRIFT;
// the due particles counted per block).  The first thread adds the force
// call's accepted pairs to the period's total.  (As kernels of their own with
// one atomic per wave on the count these took 37 us per sub-step of 110592
// particles, 22 of them in the counting; 7 us together.)
template <bool KICK, bool DRIFT>
__global__ void k_kdk_advance(double *__restrict__ pos, double *__restrict__ vel,
                              const double *__restrict__ acc, uint8_t *__restrict__ due, int n,
                              int t, KdkArgs k, double tau, double box,
                              uint8_t *__restrict__ rung, int *__restrict__ t_q,
                              int *__restrict__ t_next, int *__restrict__ n_due,
                              const Counters *__restrict__ counters,
                              unsigned long long *__restrict__ pairs) {
    __shared__ int cnt;
    if (threadIdx.x == 0) {
        cnt = 0;
        if (KICK && blockIdx.x == 0) {
            unsigned long long sum = 0;
            for (int c = 0; c < kCounterCopies; ++c) sum += counters[c * kCounterStride].interactions;
            *pairs += sum;
        }
    }
    if (DRIFT) __syncthreads();
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    bool next = false;
    if (i < n) {
        double v[3];
        for (int d = 0; d < 3; ++d) v[d] = vel[3 * (size_t)i + d];
        if (KICK && due[i]) {
            kick(v, acc, i, t, k, rung, t_q, t_next);
            for (int d = 0; d < 3; ++d) vel[3 * (size_t)i + d] = v[d];
        }
        if (DRIFT) {
            for (int d = 0; d < 3; ++d) {
                double x = pos[3 * (size_t)i + d] + v[d] * tau;
                double r = fmod(x, box);
                if (r < 0.0) r += box;
                if (r >= box) r -= box;
                pos[3 * (size_t)i + d] = r;
            }
            next = t_next[i] == t + 2;
            due[i] = (uint8_t)next;
        }
    }
    if (DRIFT) {
        const unsigned long long b = __ballot(next);
        if (b && (threadIdx.x & (kWave - 1)) == 0) atomicAdd(&cnt, __popcll(b));
        __syncthreads();
        if (threadIdx.x == 0 && cnt) atomicAdd(n_due, cnt);
    }
}

// y += a x over n x 3 values (long-range kicks; summing the two force halves)
__global__ void k_axpy3(double *__restrict__ vel, const double *__restrict__ acc, size_t n3,
                        double dk) {
    const size_t j = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n3) return;
    vel[j] = vel[j] + acc[j] * dk;
}

// The first force call's accepted pairs (the sum of its counter copies).
__global__ void k_kdk_accum(const Counters *__restrict__ c, unsigned long long *__restrict__ total) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        unsigned long long s = 0;
        for (int k = 0; k < kCounterCopies; ++k) s += c[k * kCounterStride].interactions;
        *total += s;
    }
}

unsigned blocks(size_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_kdk_assign(const double *acc, int n, const KdkArgs &k, uint8_t *rung,
                             int *census, hipStream_t s) {
    if (n == 0) return hipSuccess;
    k_kdk_assign<<<(unsigned)((n + 1023) / 1024), 1024, 0, s>>>(acc, n, k, rung, census);
    return hipGetLastError();
}

hipError_t launch_kdk_first(double *vel, const double *acc, int n, const KdkArgs &k,
                            const uint8_t *rung, int *t_q, int *t_next, hipStream_t s) {
    if (n == 0) return hipSuccess;
    k_kdk_first<<<blocks(n), 256, 0, s>>>(vel, acc, n, k, rung, t_q, t_next);
    return hipGetLastError();
}

hipError_t launch_kdk_advance(const KdkAdvance &a, bool kick, bool drift, int t, const KdkArgs &k,
                              int *n_due, hipStream_t s) {
    if (a.n == 0) return hipSuccess;
    auto fn = !kick ? k_kdk_advance<false, true>
              : drift ? k_kdk_advance<true, true>
                      : k_kdk_advance<true, false>;
    fn<<<(unsigned)((a.n + 1023) / 1024), 1024, 0, s>>>(a.pos, a.vel, a.acc, a.due, a.n, t, k, a.tau,
                                                       a.box, a.rung, a.t_q, a.t_next, n_due,
                                                       a.counters, a.pairs);
    return hipGetLastError();
}

hipError_t launch_axpy3(double *vel, const double *acc, int n, double dk, hipStream_t s) {
    if (n == 0) return hipSuccess;
    k_axpy3<<<blocks(3 * (size_t)n), 256, 0, s>>>(vel, acc, 3 * (size_t)n, dk);
    return hipGetLastError();
}

hipError_t launch_kdk_accum(const Counters *c, unsigned long long *total, hipStream_t s) {
    k_kdk_accum<<<1, 64, 0, s>>>(c, total);
    return hipGetLastError();
}

}  // namespace p3m
