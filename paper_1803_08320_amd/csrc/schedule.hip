// Work orders for the persistent adaptive kernel: by expected length (what the integrator
// uses), and by periapsis.
//
// An adaptive integrator spends most of its attempts near the orbit's closest approach,
// so the lanes of one batch need very different numbers of attempts (a factor ~10
// between the 10% and the 100% quantiles on bound Kerr orbits).  The persistent work
// queue hands lanes out in the order it is given; a lane that is long and handed out
// late keeps its wavefront busy after every other has drained the queue.  Handing the
// longest lanes out first (the longest-processing-time rule) removes that tail.
// MALBEC_SCHED_PERIAPSIS, named after its first form, ranks the lanes by their expected
// length until tau_end (sched_cost_kernel below).  malbec_adaptive_order ranks them by the
// periapsis r_p alone, read off the Carter-separated radial equation of the lane's own
// constants (E, L_z, Q, mu^2) (Sections 3-4 integrate the same constants of motion):
//   (rho^2 dr/dtau)^2 = R(r) = [E (r^2 + a^2) - a L_z]^2 - Delta [mu^2 r^2 + (L_z - a E)^2 + Q],
// R(r_0) >= 0 at the lane's radius; r_p is the first zero of R inward from r_0.
//
// The periapsis key of lane i is the bucket j of r_p on the grid r_j = r_+ 2^(j/32) (2.2% wide):
// the largest j <= j_0 (r_j <= r_0) with R(r_j) < 0, found by a march inward one bucket
// at a time (a coarser march can step over the forbidden band of an orbit close to
// marginal stability, whose periapsis is small and whose lane is long).  R(r_+) >= 0
// always (Delta = 0 there), so a lane whose R stays >= 0 down to r_+ plunges (or has a
// band narrower than a bucket); it gets key 0 and goes first with the smallest periapses,
// which costs little when the lane is short and avoids handing out a long one last.
// Every lane the integrator will not load (not ACTIVE, tau >= tau_end, bad spacetime
// index) gets the last key, MALBEC_SCHED_BUCKETS - 1.  The order
// is a counting sort of the keys (a histogram, its exclusive scan, and a scatter that
// ranks the lanes of one block in LDS and reserves their slots with one atomic per
// bucket).  Within a bucket the order depends on the timing of those atomics; the
// integration of a lane does not depend on when it is handed out.
#include "internal.hpp"
#include "monitor.hpp"

namespace malbec {

namespace {

constexpr int kBins = MALBEC_SCHED_BUCKETS;  // 1024
constexpr double kPerOctave = 32.0;

struct KeyArgs {
    int64_t n;
    const double *state;
    const double *tau;
    const int32_t *status;
    const int32_t *st_of_lane;
    double tau_end;
    uint32_t *key;
};

struct RadialPotential {
    double M, a, E, L, Q, mu2;
    __device__ __forceinline__ double operator()(double r) const
    {
        const double r2a2 = r * r + a * a;
        const double Delta = r2a2 - 2.0 * M * r;
        const double P = E * r2a2 - a * L;
        const double K = L - a * E;
        return P * P - Delta * (mu2 * r * r + K * K + Q);
    }
};

template <bool MULTI>
__global__ void __launch_bounds__(256) sched_key_kernel(KeyArgs A, StTable T)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    uint32_t key = kBins - 1;
    int32_t sid = 0;
    bool ok = A.status[i] == kActive && A.tau[i] < A.tau_end;
    if (MULTI) {
        sid = A.st_of_lane[i];
        ok = ok && sid >= 0 && sid < T.n_st;
    }
    if (ok) {
        const Spacetime S = T.st[MULTI ? sid : 0];
        double y[8], I[4];
#pragma unroll
        for (int k = 0; k < 8; ++k) y[k] = A.state[k * A.n + i];
        lane_invariants<false>(S.M, S.a, y, I);
        const RadialPotential R{S.M, S.a, I[0], I[1], I[2], -I[3]};
        const double rp = S.M + sqrt(fmax(S.M * S.M - S.a * S.a, 0.0));
        const double x = kPerOctave * log2(y[1] / rp);  // NaN, +-inf and r_0 <= r_+ fail the test
        if (x >= 1.0 && __builtin_isfinite(R.E) && __builtin_isfinite(R.L) && __builtin_isfinite(R.Q)) {
            int j = (int)fmin(x, (double)(kBins - 2));
            while (j > 0 && !(R(rp * exp2((double)j / kPerOctave)) < 0.0)) --j;
            key = (uint32_t)j;  // j = 0: no turning point above r_+
        }
    }
    A.key[i] = key;
}

// Key of lane i by its expected length (longest first), from the Mino time lambda
// (dtau = rho^2 dlambda) that it runs through until tau_end.  In lambda the radial motion of
// Carter's separation is that of a particle in a quartic potential, (dr/dlambda)^2 = R(r),
// d^2 r / dlambda^2 = R'(r) / 2, and an adaptive step, about r^(7/4) in tau, is nearly
// constant in lambda.  The radial motion is followed in single precision (rho^2 taken as r^2,
// lengths in units of M) with steps of kStep r^(-5/4), dr/dlambda put back on R after each step that
// does not turn (which keeps an orbit next to the separatrix on its side of the barrier: without
// it 1.5 % of the benchmark's orbits seemed to plunge, and they are among the longest), until
// tau_end, the stop radius or the escape radius; after kMaxSteps of them the rest is
// extrapolated.  The attempts of the benchmark's orbits (a = 0.9 and 0.3, tau = 400, tolerances
// 1e-10 and 1e-12) follow lambda^0.82 L_z^-0.47 (mu^2 - E^2)^-0.35 within 6.4 % rms and at most 15 %
// upwards (a small L_z means a passage near the axis); the periapsis correlates with them
// at 0.48 (the exponents are fitted to these orbits; other batches get another order, never another
// result, and gain as well: null, unbound and near-equatorial orbits, spins 0 to 0.998, tolerances 1e-6
// and 1e-9 take 1 to 38 % less time than in the order by periapsis, alone 200,000 and 262,144 orbits close to
// circular, 8 < r < 16, take 7 to 9 % more).  Bound by the steps' single-precision arithmetic: 64 us for 262,144 lanes.  The
// integration in this order against that by periapsis, on one MI355X (tau = 400, 1e-12):
// 65,536 lanes 5.4 -> 4.6 ms, 262,144 lanes 7.7 -> 5.3 ms, 1,048,576 lanes 15.4 -> 13.8 ms,
// and 9.8 -> 6.6 ms for 262,144 lanes at a = 0.3, a quarter of which plunge.
constexpr float kStep = 0.8f, kStepMax = 0.1f;
constexpr int kMaxSteps = 256;
template <bool MULTI>
__global__ void __launch_bounds__(256) sched_cost_kernel(KeyArgs A, StTable T, double r_escape)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    uint32_t key = kBins - 1;
    int32_t sid = 0;
    const double tau0 = A.tau[i];
    bool ok = A.status[i] == kActive && tau0 < A.tau_end;
    if (MULTI) {
        sid = A.st_of_lane[i];
        ok = ok && sid >= 0 && sid < T.n_st;
    }
    if (ok) {
        const Spacetime S = T.st[MULTI ? sid : 0];
        double y[8], I[4];
#pragma unroll
        for (int k = 0; k < 8; ++k) y[k] = A.state[k * A.n + i];
        lane_invariants<false>(S.M, S.a, y, I);
        const double iM = 1.0 / S.M, a = S.a * iM, E = I[0], L = I[1] * iM, Q = I[2] * iM * iM, mu2 = -I[3];
        const double K = (L - a * E) * (L - a * E) + Q;
        // R = c4 r^4 + c3 r^3 + c2 r^2 + c1 r + c0; R'/2 and R''/2
        const float c4 = (float)(E * E - mu2), c3 = (float)(2.0 * mu2),
                    c2 = (float)(a * a * (E * E - mu2) - L * L - Q), c1 = (float)(2.0 * K),
                    c0 = (float)(-a * a * Q);
        float r = (float)(y[1] * iM);
        const double c = cos(y[2]);
        float v = (float)((y[1] * y[1] * iM * iM + a * a * c * c) * y[5]);  // dr/dlambda
        const float r_stop = (float)(S.r_stop * iM), r_esc = (float)(r_escape * iM);
        const float tau_end = (float)((A.tau_end - tau0) * iM);
        float tau = 0.0f, lam = 0.0f;
        bool on = true;
        for (int k = 0; k < kMaxSteps && on; ++k) {
            const float q = __builtin_amdgcn_rsqf(r);
            const float dl = fminf(kStep * q * q * __builtin_amdgcn_sqrtf(q), kStepMax);
            auto acc = [&](float x) { return 0.5f * (((4.0f * c4 * x + 3.0f * c3) * x + 2.0f * c2) * x + c1); };
            const float ac = acc(r), jerk = 0.5f * ((12.0f * c4 * r + 6.0f * c3) * r + 2.0f * c2) * v;
            const float rn = r + dl * (v + dl * (0.5f * ac + dl * jerk * (1.0f / 6.0f)));
            float vn = v + 0.5f * dl * (ac + acc(rn));
            const float rm = 0.5f * (r + rn) - 0.125f * dl * (vn - v);
            const float dt = dl * (r * r + 4.0f * rm * rm + rn * rn) * (1.0f / 6.0f);
            const float R = (((c4 * rn + c3) * rn + c2) * rn + c1) * rn + c0;
            if (R > 0.0f && vn * v > 0.0f) vn = copysignf(__builtin_amdgcn_sqrtf(R), vn);
            const bool last = !(tau + dt < tau_end);
            lam += last ? dl * (tau_end - tau) / dt : dl;
            tau += dt;
            r = rn;
            v = vn;
            on = !last && r > r_stop && r < r_esc;
        }
        if (on) lam *= tau_end / tau;
        // attempts ~ lambda^0.82 L_z^-0.47 (mu^2 - E^2)^-0.35
        const float L2 = (float)fmax(L * L, 1e-3 * (L * L + fabs(Q))), B = (float)fmin(fmax(mu2 - E * E, 0.01), 1.0);
        const float cost = 0.82f * __builtin_amdgcn_logf(lam) - 0.235f * __builtin_amdgcn_logf(L2) -
                           0.35f * __builtin_amdgcn_logf(B);
        // 32 buckets per octave, longest first; NaN (an unusable state) goes last
        const float x = 448.0f - 32.0f * cost;
        key = x < 0.0f ? 0u : x < (float)(kBins - 2) ? (uint32_t)x : (uint32_t)(kBins - 2);
    }
    A.key[i] = key;
}

__global__ void zero_u32_kernel(uint32_t *p, int m)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < m) p[k] = 0u;
}

// count[b] += number of keys equal to b (LDS histogram per block, grid-stride).
__global__ void __launch_bounds__(256) sched_hist_kernel(const uint32_t *key, int64_t n,
                                                          uint32_t *count)
{
    __shared__ uint32_t h[kBins];
    for (int k = threadIdx.x; k < kBins; k += blockDim.x) h[k] = 0u;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&h[min(key[i], (uint32_t)(kBins - 1))], 1u);
    __syncthreads();
    for (int k = threadIdx.x; k < kBins; k += blockDim.x)
        if (h[k]) atomicAdd(&count[k], h[k]);
}

// next[b] = sum of count[b'] over b' < b (one block of kBins threads, Hillis-Steele).
__global__ void __launch_bounds__(kBins) sched_scan_kernel(const uint32_t *count, uint32_t *next)
{
    __shared__ uint32_t v[2][kBins];
    const int t = threadIdx.x;
    int cur = 0;
    v[0][t] = t > 0 ? count[t - 1] : 0u;
    __syncthreads();
    for (int d = 1; d < kBins; d <<= 1) {
        v[cur ^ 1][t] = v[cur][t] + (t >= d ? v[cur][t - d] : 0u);
        __syncthreads();
        cur ^= 1;
    }
    next[t] = v[cur][t];
}

// order[next[b] ...] = the lanes with key b.  Each block takes 256 consecutive lanes at
// a time: LDS ranks within the block, one global atomic per non-empty bucket.
__global__ void __launch_bounds__(256) sched_scatter_kernel(const uint32_t *key, int64_t n,
                                                             uint32_t *next, uint32_t *order)
{
    __shared__ uint32_t cnt[kBins];
    __shared__ uint32_t base[kBins];
    const int64_t n_chunks = (n + 255) / 256;
    for (int64_t chunk = blockIdx.x; chunk < n_chunks; chunk += gridDim.x) {
        for (int k = threadIdx.x; k < kBins; k += 256) cnt[k] = 0u;
        __syncthreads();
        const int64_t i = chunk * 256 + threadIdx.x;
        const bool in = i < n;
        const uint32_t b = in ? min(key[i], (uint32_t)(kBins - 1)) : 0u;
        const uint32_t rank = in ? atomicAdd(&cnt[b], 1u) : 0u;
        __syncthreads();
        for (int k = threadIdx.x; k < kBins; k += 256)
            if (cnt[k]) base[k] = atomicAdd(&next[k], cnt[k]);
        __syncthreads();
        if (in) order[base[b] + rank] = (uint32_t)i;
        __syncthreads();
    }
}

}  // namespace

SchedLayout sched_layout(int64_t n)
{
    SchedLayout L;
    L.count = 0;
    L.next = (size_t)kBins * sizeof(uint32_t);
    L.key = 2 * L.next;
    L.order = L.key + (((size_t)n * sizeof(uint32_t) + 255) / 256) * 256;
    L.bytes = L.order + (size_t)n * sizeof(uint32_t);
    return L;
}

int launch_adaptive_order(const StTable &T, const int32_t *st_of_lane, int64_t n,
                          const double *state, const double *tau, const int32_t *status,
                          double tau_end, uint32_t *order, uint32_t *keys, void *ws,
                          hipStream_t s, const double *by_cost_r_escape)
{
    if (n == 0) return MALBEC_OK;
    const SchedLayout Ly = sched_layout(n);
    char *w = (char *)ws;
    uint32_t *count = (uint32_t *)(w + Ly.count);
    uint32_t *next = (uint32_t *)(w + Ly.next);
    uint32_t *key = keys ? keys : (uint32_t *)(w + Ly.key);
    const bool multi = st_of_lane != nullptr && T.n_st > 1;
    KeyArgs A{n, state, tau, status, multi ? st_of_lane : nullptr, tau_end, key};
    if (by_cost_r_escape && multi)
        hipLaunchKernelGGL((sched_cost_kernel<true>), dim3(grid_for(n, 256)), dim3(256), 0, s, A, T,
                           *by_cost_r_escape);
    else if (by_cost_r_escape)
        hipLaunchKernelGGL((sched_cost_kernel<false>), dim3(grid_for(n, 256)), dim3(256), 0, s, A, T,
                           *by_cost_r_escape);
    else if (multi)
        hipLaunchKernelGGL((sched_key_kernel<true>), dim3(grid_for(n, 256)), dim3(256), 0, s, A, T);
    else
        hipLaunchKernelGGL((sched_key_kernel<false>), dim3(grid_for(n, 256)), dim3(256), 0, s, A, T);
    MALBEC_LAUNCH_CHECK("sched_key_kernel");
    hipLaunchKernelGGL(zero_u32_kernel, dim3(kBins / 256), dim3(256), 0, s, count, kBins);
    MALBEC_LAUNCH_CHECK("zero_u32_kernel");
    const unsigned g = (unsigned)std::min<int64_t>(grid_for(n, 256), 1024);
    hipLaunchKernelGGL(sched_hist_kernel, dim3(g), dim3(256), 0, s, key, n, count);
    MALBEC_LAUNCH_CHECK("sched_hist_kernel");
    hipLaunchKernelGGL(sched_scan_kernel, dim3(1), dim3(kBins), 0, s, count, next);
    MALBEC_LAUNCH_CHECK("sched_scan_kernel");
    hipLaunchKernelGGL(sched_scatter_kernel, dim3(g), dim3(256), 0, s, key, n, next, order);
    MALBEC_LAUNCH_CHECK("sched_scatter_kernel");
    return MALBEC_OK;
}

}  // namespace malbec
