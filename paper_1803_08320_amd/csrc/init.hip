// Initial-condition construction on the device, one thread per lane (the CONSTANTS
// sampler: one wavefront for a run of lanes, see sample_kernel).
//
//  CANONICAL  the paper's IC table rows (t, r, theta, phi, p_t, p_r, p_theta, p_phi)
//             with p_t = +E (Section 5); u^mu = g^{mu nu} p_nu with p_t -> -E.
//  CIRCULAR   equatorial circular orbits (Sections 3-4) in the Bardeen-Press-
//             Teukolsky form, with a seeded relative perturbation of L.
//  CONSTANTS  seeded (r0, theta0, E, L_z, Q, signs) accepted when Carter's radial
//             and polar potentials are non-negative; u from the separated equations.
// Random numbers: SplitMix64 (Steele, Lea & Flood 2014) used as a counter-based
// generator, draw k of attempt j of lane i = output (i*2^24 + j*2^4 + k + 1) of the
// sequence started at `seed`.
#include <mutex>

#include "ic_device.hpp"
#include "internal.hpp"

namespace malbec {

namespace {

__device__ __forceinline__ uint64_t splitmix_out(uint64_t seed, uint64_t lane, uint64_t attempt,
                                                 uint64_t k)
{
    uint64_t z = seed + (((lane << 24) | (attempt << 4) | k) + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ double unit53(uint64_t x) { return (double)(x >> 11) * 0x1.0p-53; }

// lo + (hi - lo) u, rounded after each operation (no fused multiply-add), so that
// the drawn values are the same bits on every implementation of the recipe.
__device__ __forceinline__ double uniform(const double rg[2], uint64_t x)
{
#pragma clang fp contract(off)
    const double span = rg[1] - rg[0];
    const double scaled = span * unit53(x);
    return rg[0] + scaled;
}

// dL (2u - 1) with separately rounded operations.
__device__ __forceinline__ double centred(double dL, uint64_t x)
{
#pragma clang fp contract(off)
    const double twice = 2.0 * unit53(x);
    return dL * (twice - 1.0);
}

struct InitArgs {
    malbec_ic_spec spec;
    const int32_t *st_of_lane;
    int64_t n;
    double *state;
    double *consts;
    int64_t *attempts;
    unsigned long long *exhausted;  // strict mode: count of lanes that exhausted the sampler
};

// Lanes whose rejection sampler ran out of attempts in a strict call (one counter per
// GPU: each device holds its own copy, found through hipGetSymbolAddress).
__device__ unsigned long long g_exhausted;

__global__ void zero_exhausted_kernel(unsigned long long *p) { *p = 0ull; }

// The outputs of lane i (nan: a state that could not be formed).
__device__ __forceinline__ void store_lane(const InitArgs &A, int64_t i, bool nan, const double y[8],
                                           double E, double L, double Q, double mu2, int64_t used)
{
#pragma unroll
    for (int k = 0; k < 8; ++k) A.state[k * A.n + i] = nan ? __builtin_nan("") : y[k];
    if (A.consts) {
        A.consts[0 * A.n + i] = E;
        A.consts[1 * A.n + i] = L;
        A.consts[2 * A.n + i] = Q;
        A.consts[3 * A.n + i] = mu2;
    }
    if (A.attempts) A.attempts[i] = used;
}

__global__ void __launch_bounds__(256) init_kernel(InitArgs A, StTable T)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    int32_t sid = A.st_of_lane ? A.st_of_lane[i] : 0;
    const bool bad_sid = sid < 0 || sid >= T.n_st;  // invalid index: NaN state
    if (bad_sid) sid = 0;
    const Spacetime S = T.st[sid];
    const double M = S.M, a = S.a;
    const malbec_ic_spec &P = A.spec;
    const uint64_t lane = (uint64_t)(P.lane0 + i);
    double y[8];
    double cE = 0.0, cL = 0.0, cQ = 0.0, cmu2 = P.mu2;

    if (P.mode == MALBEC_IC_CANONICAL) {
        const double *z = P.rows + 8 * i;
        double s, c;
        sincos(z[2], &s, &c);
        double itt, itp, ipp, irr, ithth;
        inverse_metric(M, a, z[1], s, c, itt, itp, ipp, irr, ithth);
        const double pt = -z[4];
        y[0] = z[0]; y[1] = z[1]; y[2] = z[2]; y[3] = z[3];
        y[4] = itt * pt + itp * z[7];
        y[5] = irr * z[5];
        y[6] = ithth * z[6];
        y[7] = itp * pt + ipp * z[7];
        cE = z[4];
        cL = z[7];
        cmu2 = 1.0;
    } else if (P.mode == MALBEC_IC_PARAMS) {
        const double *z = P.rows + 6 * i;  // r0, theta0, u^r0, u^theta0, L_z, E
        double s, c;
        sincos(z[1], &s, &c);
        double itt, itp, ipp, irr, ithth;
        inverse_metric(M, a, z[0], s, c, itt, itp, ipp, irr, ithth);
        y[0] = 0.0; y[1] = z[0]; y[2] = z[1]; y[3] = 0.0;
        y[4] = itt * (-z[5]) + itp * z[4];
        y[5] = z[2];
        y[6] = z[3];
        y[7] = itp * (-z[5]) + ipp * z[4];
        cE = z[5];
        cL = z[4];
        cmu2 = 1.0;
    } else {  // MALBEC_IC_CIRCULAR
        const double rg[2] = {P.r_lo, P.r_hi};
        const double r0 = uniform(rg, splitmix_out(P.seed, lane, 0, 0));
        const double delta = centred(P.dL, splitmix_out(P.seed, lane, 0, 1));
        // Bardeen-Press-Teukolsky circular orbit, upper sign prograde
        const double sg = P.prograde ? 1.0 : -1.0;
        const double sr = sqrt(r0), sM = sqrt(M);
        const double den = pow(r0, 0.75) * sqrt(r0 * sr - 3.0 * M * sr + sg * 2.0 * a * sM);
        const double Ec = (r0 * sr - 2.0 * M * sr + sg * a * sM) / den;
        const double Lc = sg * sM * (r0 * r0 - sg * 2.0 * a * sM * sr + a * a) / den;
        const double L = Lc * (1.0 + delta);
        double itt, itp, ipp, irr, ithth;
        inverse_metric(M, a, r0, 1.0, 0.0, itt, itp, ipp, irr, ithth);
        double E = Ec;
        if (P.e_from_norm) {
            // g^{mu nu} p_mu p_nu = -1 with p = (-E, 0, 0, L): quadratic in E, g^tt < 0
            const double qa = itt, qb = -2.0 * itp * L, qc = ipp * L * L + 1.0;
            E = (-qb - sqrt(qb * qb - 4.0 * qa * qc)) / (2.0 * qa);
        }
        y[0] = 0.0; y[1] = r0; y[2] = 1.57079632679489661923; y[3] = 0.0;
        y[4] = itt * (-E) + itp * L;
        y[5] = 0.0;
        y[6] = 0.0;
        y[7] = itp * (-E) + ipp * L;
        cE = E;
        cL = L;
        cQ = 0.0;
        cmu2 = 1.0;
    }
    store_lane(A, i, bad_sid, y, cE, cL, cQ, cmu2, 1);
}

// ---- the CONSTANTS sampler ------------------------------------------------------------
// One attempt's draws.
struct Draw {
    double r, th, E, L, Q;
};
__device__ __forceinline__ Draw draw_attempt(const malbec_ic_spec &P, uint64_t lane, uint64_t att)
{
    Draw D;
    D.r = uniform(P.r_range, splitmix_out(P.seed, lane, att, 0));
    D.th = uniform(P.th_range, splitmix_out(P.seed, lane, att, 1));
    D.E = uniform(P.E_range, splitmix_out(P.seed, lane, att, 2));
    D.L = uniform(P.Lz_range, splitmix_out(P.seed, lane, att, 3));
    D.Q = uniform(P.Q_range, splitmix_out(P.seed, lane, att, 4));
    return D;
}

// R(r) >= 0 and Theta(theta) >= 0.  The sign of Theta comes from Theta sin^2 theta (no division) where that is
// clear of its own rounding and of that of sincos_any (1e-16 of the terms without their factor cos^2;
// its reduction holds for |theta| < 1e6), elsewhere from the expression that the lane's state is formed
// with, so that a draw on the boundary is decided as its state will have it.
// big_theta: a range beyond sincos_any.
__device__ __forceinline__ bool admissible(const malbec_ic_spec &P, double M, double a, const Draw &D,
                                           bool big_theta)
{
    const double R = radial_potential(M, a, D.E, D.L, D.Q, P.mu2, D.r);
    if (!(R >= 0.0)) return false;
    double s, c;
    bool ok = false, close = true;
    if (!big_theta) {
        sincos_any(D.th, s, c);
        const double s2 = s * s, c2 = c * c, LL = D.L * D.L;
        const double Qs = D.Q * s2, k = a * a * (P.mu2 - D.E * D.E) * s2;
        const double T = Qs - c2 * (k + LL);
        ok = T > 0.0;
        close = !(fabs(T) > 1e-10 * (fabs(Qs) + (fabs(k) + LL)));
    }
    if (close) {
        sincos(D.th, &s, &c);
        ok = polar_potential(a, D.E, D.L, D.Q, P.mu2, s, c) >= 0.0;
    }
    return ok;
}

// A lane takes as many attempts as it needs (20 on the average for the benchmark's ranges,
// at an acceptance of 5 %), so a wavefront with one lane per thread waits for the slowest
// of 64 (95 attempts).  Here a wavefront works through a run of `run` lanes: a thread
// whose lane is settled takes the next one of the run, and when the run is used up the
// threads left over help: with P lanes pending, g = 64 / P threads (a power of two) try g
// consecutive attempts of each, and the first that is admissible counts.  (The generator
// is counter-based: attempt j of lane i needs no earlier draw.)  The search settles only
// the attempt of each lane, kept in LDS; then the wavefront forms the states of its run,
// 64 at a time, with all threads busy and coalesced stores.
// Bound by VALU issue (0.84 of the time; about 245 instructions per attempt, half of them
// the generator's).  Measured on one MI355X with 1,048,576 lanes of the benchmark's ranges,
// against one thread per lane: 705 -> 195 us, 3.35 x 10^8 -> 0.89 x 10^8 wavefront
// instructions.  Where nearly every draw is admissible, 16,384 to 100,000 lanes take 2 to 5 us more than with
// one thread per lane (18-21 us): a run is shorter than a wavefront and has no attempts to share; runs
// of 32 and 64 lanes would cost the benchmark's ranges as much or more.
constexpr int kMaxRun = 256;     // lanes per wavefront: their attempts' LDS
constexpr int kSampleBlock = 256;
template <bool MULTI>
__global__ void __launch_bounds__(kSampleBlock) sample_kernel(InitArgs A, StTable T, int32_t run,
                                                              bool big_theta)
{
    constexpr int kWaves = kSampleBlock / 64;
    __shared__ Spacetime lds_st[MULTI ? kMaxSt : 1];
    __shared__ int32_t lds_att[kWaves][kMaxRun];  // admissible attempt of each lane of the run
    __shared__ int32_t lds_src[kWaves][64];       // thread that holds pending lane number k
    if (MULTI) {
        for (int k = threadIdx.x; k < T.n_st; k += blockDim.x) lds_st[k] = T.st[k];
        __syncthreads();
    }
    const malbec_ic_spec &P = A.spec;
    const int t = (int)(threadIdx.x & 63u), w = (int)(threadIdx.x >> 6);
    const int64_t first = ((int64_t)blockIdx.x * kWaves + w) * run;
    if (first >= A.n) return;
    const int32_t len = (int32_t)(A.n - first < run ? A.n - first : run);
    const int32_t max_att = (int32_t)P.max_attempts;
    auto spacetime_of = [&](int64_t i, bool &bad) {
        const int32_t s = MULTI ? A.st_of_lane[i] : 0;
        bad = s < 0 || s >= T.n_st;  // invalid index: sampled as spacetime 0, NaN state
        return bad ? 0 : s;
    };

    int32_t next = 0;             // first lane of the run that no thread has taken (uniform)
    int32_t item = -1, att = 0, sid = 0;  // this thread's lane of the run and its next attempt
    for (;;) {
        const unsigned long long idle = __ballot(item < 0);
        if (idle != 0ull && next < len) {
            const int rank = (int)__builtin_amdgcn_mbcnt_hi(
                (unsigned)(idle >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)idle, 0u));
            if (item < 0 && next + rank < len) {
                bool bad;
                item = next + rank;
                att = 0;
                sid = spacetime_of(first + item, bad);
            }
            const int32_t up = next + __popcll(idle);
            next = up < len ? up : len;
        }
        const unsigned long long pending = __ballot(item >= 0);
        if (pending == 0ull) break;
        const int n_pend = __popcll(pending);
        const int sh = n_pend > 32 ? 0 : n_pend > 16 ? 1 : n_pend > 8 ? 2 : n_pend > 4 ? 3
                       : n_pend > 2 ? 4 : n_pend > 1 ? 5 : 6;  // 2^sh attempts of each
        const int my = (int)__builtin_amdgcn_mbcnt_hi(
            (unsigned)(pending >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)pending, 0u));
        if (n_pend < 64 && item >= 0) lds_src[w][my] = t;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        int32_t try_item = item, try_att = att, try_sid = sid;
        if (n_pend < 64) {
            const int group = t >> sh;
            const int src = group < n_pend ? lds_src[w][group] : t;
            try_item = __shfl(item, src, 64);
            try_att = __shfl(att, src, 64) + (t & ((1 << sh) - 1));
            if (MULTI) try_sid = __shfl(sid, src, 64);
            if (group >= n_pend) try_att = max_att;  // nothing to try
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        bool ok = false;
        if (try_att < max_att) {
            const Spacetime S = MULTI ? lds_st[try_sid] : T.st[0];
            const Draw D = draw_attempt(P, (uint64_t)(P.lane0 + first + try_item), (uint64_t)try_att);
            ok = admissible(P, S.M, S.a, D, big_theta);
        }
        const unsigned long long hits = __ballot(ok);
        if (item >= 0) {
            // the attempts of this thread's lane were made by threads my 2^sh ... + 2^sh - 1
            const unsigned long long mine = (hits >> ((my << sh) & 63)) &
                                            (sh == 6 ? ~0ull : (1ull << (1 << sh)) - 1ull);
            if (mine != 0ull) {
                lds_att[w][item] = att + __ffsll((long long)mine) - 1;
                item = -1;
            } else {
                att += 1 << sh;
                if (att >= max_att) {
                    lds_att[w][item] = max_att;  // none admissible
                    item = -1;
                }
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int32_t k = t; k < len; k += 64) {
        const int64_t i = first + k;
        bool bad;
        const int32_t k_st = spacetime_of(i, bad);
        const Spacetime S = MULTI ? lds_st[k_st] : T.st[0];
        const uint64_t lane = (uint64_t)(P.lane0 + i);
        const bool found = lds_att[w][k] < max_att;
        const int32_t j = found ? lds_att[w][k] : max_att - 1;
        const Draw D = draw_attempt(P, lane, (uint64_t)j);
        const double sr = (splitmix_out(P.seed, lane, (uint64_t)j, 5) >> 63) ? -1.0 : 1.0;
        const double sth = (splitmix_out(P.seed, lane, (uint64_t)j, 6) >> 63) ? -1.0 : 1.0;
        double s, c;
        sincos(D.th, &s, &c);
        const double R = radial_potential(S.M, S.a, D.E, D.L, D.Q, P.mu2, D.r);
        const double Th = polar_potential(S.a, D.E, D.L, D.Q, P.mu2, s, c);
        double y[8] = {0.0, D.r, D.th, 0.0, 0.0, 0.0, 0.0, 0.0};
        velocity(S.M, S.a, D.E, D.L, D.Q, P.mu2, D.r, s, c, sr, sth, R, Th, y + 4);
        if (!found && A.exhausted) atomicAdd(A.exhausted, 1ull);
        store_lane(A, i, bad || !found, y, D.E, D.L, D.Q, P.mu2, found ? j + 1 : max_att);
    }
}

}  // namespace

// The device address of g_exhausted on the current device, looked up once per device
// (each GPU holds its own copy at its own address; the name itself is a host-side
// stand-in that must not be passed to a kernel).
static int exhausted_counter(unsigned long long **out)
{
    constexpr int kDevices = 64;
    static std::mutex mu;
    static unsigned long long *ptr[kDevices] = {};
    int dev = 0;
    MALBEC_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kDevices)
        return fail(MALBEC_ENOTSUP, "device %d: the strict sampler count covers %d devices", dev, kDevices);
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        MALBEC_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(g_exhausted)));
        if (!p) return fail(MALBEC_EDEVICE, "hipGetSymbolAddress returned NULL for the sampler count");
        ptr[dev] = (unsigned long long *)p;
    }
    *out = ptr[dev];
    return MALBEC_OK;
}

int launch_init(const malbec_ic_spec &spec, const StTable &T, const int32_t *st_of_lane, int64_t n,
                double *state, double *consts, int64_t *attempts, hipStream_t s)
{
    InitArgs A;
    A.spec = spec;
    A.st_of_lane = T.n_st > 1 ? st_of_lane : nullptr;
    A.n = n;
    A.state = state;
    A.consts = consts;
    A.attempts = attempts;
    A.exhausted = nullptr;
    const bool strict = spec.strict != 0 && spec.mode == MALBEC_IC_CONSTANTS;
    if (strict) {
        int rc = exhausted_counter(&A.exhausted);
        if (rc) return rc;
        hipLaunchKernelGGL(zero_exhausted_kernel, dim3(1), dim3(1), 0, s, A.exhausted);
        MALBEC_LAUNCH_CHECK("zero_exhausted_kernel");
    }
    if (spec.mode == MALBEC_IC_CONSTANTS) {
        // As many wavefronts as the chip holds (256 CUs x 16 at the kernel's registers), each
        // with as short a run of lanes as that leaves: a batch below 2^18 lanes has several
        // threads per lane from the start.
        constexpr int64_t kWavesOfChip = 4096;
        const int64_t want = (n + kWavesOfChip - 1) / kWavesOfChip;
        const int32_t run = (int32_t)(want < kMaxRun ? want : kMaxRun);
        const int64_t waves = (n + run - 1) / run;
        const bool big_theta = fmax(fabs(spec.th_range[0]), fabs(spec.th_range[1])) > 1e5;
        const dim3 grid(grid_for(waves, kSampleBlock / 64)), block(kSampleBlock);
        if (A.st_of_lane)
            hipLaunchKernelGGL((sample_kernel<true>), grid, block, 0, s, A, T, run, big_theta);
        else
            hipLaunchKernelGGL((sample_kernel<false>), grid, block, 0, s, A, T, run, big_theta);
        MALBEC_LAUNCH_CHECK("sample_kernel");
    } else {
        const int block = 256;
        hipLaunchKernelGGL(init_kernel, dim3(grid_for(n, block)), dim3(block), 0, s, A, T);
        MALBEC_LAUNCH_CHECK("init_kernel");
    }
    if (strict) {
        unsigned long long count = 0;
        MALBEC_HIP_CHECK(hipMemcpyAsync(&count, A.exhausted, sizeof(count), hipMemcpyDeviceToHost, s));
        MALBEC_HIP_CHECK(hipStreamSynchronize(s));
        if (count > 0)
            return fail(MALBEC_ESAMPLE, "%llu of %lld lanes exhausted max_attempts = %lld", count,
                        (long long)n, (long long)spec.max_attempts);
    }
    return MALBEC_OK;
}

}  // namespace malbec
