// FP64 fixed-step RK4 integrator: one lane (thread) per geodesic.
//
// Each lane loads its 8-component state once (coalesced, component-major), runs
// the steps of the launch with all stage values in registers and stores the state
// once.  The only global traffic is 64 B in + 64 B out + status/steps per lane per
// launch; the work is FP64 VALU arithmetic.  Spacetime constants come from the
// kernel arguments (uniform batch) or from an LDS copy of the table (mixed batch).
//
// What bounds them: FP64 VALU issue (0.98 of the CU-busy time on a full chip), so a step
// costs its instructions: 342 FP64 arithmetic ones and 21.5 others per Christoffel step,
// 264 and 23 per Hamiltonian step (358 and 27, 290 and 27 with the acceleration of the
// FP32-compensated kernels, sums of the stage velocities and FP64 stop tests).  Measured on
// one MI355X, the same machine before that and now:
//   1,048,576 Kerr lanes x 1,000 steps: 12.05 -> 11.4 ms (9.2 x 10^10 lane-steps/s)
//   300,007 lanes x 1,000 steps, Hamiltonian form: 3.18 -> 2.78 ms
//   1,024 Schwarzschild lanes x 2,000 steps (one wave on each of 16 SIMDs): 1.93 -> 1.43 ms
#include "checkpoint.hpp"
#include "f64_prog.hpp"
#include "internal.hpp"
#include "monitor.hpp"
#include "turns.hpp"

namespace malbec {

namespace {

__device__ __forceinline__ void put_slot(const IntArgs &A, int64_t i, int32_t slot, const double y[8])
{
    double *base = A.ckpt + (int64_t)slot * 8 * A.n;
#pragma unroll
    for (int k = 0; k < 8; ++k) base[k * A.n + i] = y[k];
}

// UNIT_M: the batch's one spacetime has M = 1 (the unit of the paper's runs), known at
// compile time, which removes the multiplications by M (exact: the results are the
// bits of the general kernel).
// ZERO_A: it has a = 0 (Schwarzschild), known at compile time, which removes the terms that are
// then zero: 48 of the 240 arithmetic instructions of a step's four Christoffel accelerations, 24
// of the Hamiltonian form's 176 (the same bits).  On one MI355X, 1,000 steps: 1,024 lanes
// 0.883 -> 0.770 ms, 262,144 lanes 2.95 -> 2.48 ms, 1,048,576 lanes 11.41 -> 9.61 ms; Hamiltonian
// form 0.756 -> 0.733, 2.40 -> 2.23 and 9.23 -> 8.59 ms.
template <bool MULTI, bool CKPT, bool HAM, bool UNIT_M = false, bool ZERO_A = false>
__global__ void __launch_bounds__(256) rk4_f64_kernel(IntArgs A, StTable T)
{
    __shared__ Spacetime lds_st[kMaxSt];
    if (MULTI) {
        for (int k = threadIdx.x; k < T.n_st; k += blockDim.x) lds_st[k] = T.st[k];
        __syncthreads();
    }
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    int32_t st = A.status[i];
    int32_t sid = 0;
    if (MULTI) {
        sid = A.st_of_lane[i];
        if (sid < 0 || sid >= T.n_st) {  // invalid spacetime index: the lane cannot step
            sid = 0;
            if (st == kActive) st = kNonfinite;
            A.status[i] = st;
        }
    }
    Spacetime S = MULTI ? lds_st[sid] : T.st[0];
    if (UNIT_M) S.M = 1.0;
    // first thread of this wavefront (wave-uniform, held in a scalar register)
    const int32_t wave0 = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x) & ~63;

    double y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) y[k] = A.state[k * A.n + i];
    const HamConst<double> P = ham_const(S.a, y[4], y[7]);
    int32_t taken = 0;
    if (!CKPT && st == kActive) {
        // a launch always has n_steps >= 1 (the launcher makes none for a call of zero steps)
        taken = run_steps<HAM, ZERO_A>(S, P, A.h, A.r_escape, A.n_steps, y, st);
        // the lane's index rebuilt from wave-uniform values and its position in the
        // wavefront: no per-lane address stays live across the loop
        const int64_t ie = (int64_t)blockIdx.x * blockDim.x + wave0 +
                           (int32_t)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll
        for (int k = 0; k < 8; ++k) A.state[k * A.n + ie] = y[k];
        A.status[ie] = st;
        A.steps[ie] += taken;
    } else if (CKPT || st == kActive) {  // (without CKPT never: the other instances keep their registers)
        const bool was_active = st == kActive;
        taken = run_checkpointed(
            A.k0, A.n_steps, A.ck_every, A.ck_last, was_active,
            [&](int32_t m, bool &active) {
                const int32_t ks = run_steps<HAM>(S, P, A.h, A.r_escape, m, y, st);
                active = st == kActive;
                return ks;
            },
            [&](int32_t slot) { put_slot(A, i, slot, y); });
        if (was_active) {
#pragma unroll
            for (int k = 0; k < 8; ++k) A.state[k * A.n + i] = y[k];
            A.status[i] = st;
            A.steps[i] += taken;
        }
    }
}

// A number of lanes that fills the chip unevenly, for instance 100,003: 1,563 wavefronts on 1,024
// SIMDs, so that half of these run two, and the other half wait for them.  Here a whole number of
// blocks per CU takes `share` >= 256 consecutive lanes each and advances 256 of them at a time by q
// steps, in turns: turn t runs the lanes t 256 .. t 256 + 255 modulo the share, so that every lane has
// its steps after (steps / q) share / 256 turns, at the same time on every SIMD.  Between its turns a lane is
// parked in LDS (72 B).  The rule for taking this launch (turns_blocks) and its measurements are in
// api.hip.
template <bool MULTI, bool HAM, bool UNIT_M, bool ZERO_A>
__global__ void __launch_bounds__(256) rk4_f64_turns_kernel(IntArgs A, StTable T, int32_t share, int32_t q)
{
    __shared__ Spacetime lds_st[MULTI ? kMaxSt : 1];
    if (MULTI)
        for (int k = threadIdx.x; k < T.n_st; k += blockDim.x) lds_st[k] = T.st[k];
    __shared__ int32_t worked;        // the last turn in which a lane stepped
    extern __shared__ double park[];  // [8][share], then status and steps taken
    int32_t *lane_st = (int32_t *)(park + 8 * share), *lane_taken = lane_st + share;
    const int64_t base = (int64_t)blockIdx.x * share;
    const int64_t rest = A.n - base;
    const int32_t m = rest < share ? (int32_t)rest : share;  // lanes of this block (may be <= 0)
    const int32_t t = (int32_t)threadIdx.x;
    if (t == 0) worked = 0;
    for (int32_t j = t; j < m; j += 256) {
        int32_t st = A.status[base + j];
        if (MULTI) {
            const int32_t sid = A.st_of_lane[base + j];
            if (sid < 0 || sid >= T.n_st) {  // invalid spacetime index: the lane cannot step
                if (st == kActive) st = kNonfinite;
                A.status[base + j] = st;
            }
        }
        lane_st[j] = st;
        lane_taken[j] = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) park[k * share + j] = A.state[k * A.n + base + j];
    }
    __syncthreads();
    Spacetime S = T.st[0];
    if (UNIT_M) S.M = 1.0;
    const int32_t turns = turns_of_block(A.n_steps, q, m);
    int32_t j = t;
    for (int32_t turn = 0; turn < turns; ++turn) {
        if (j < m && lane_st[j] == kActive && lane_taken[j] < A.n_steps) {
            const int32_t taken = lane_taken[j], left = A.n_steps - taken;
            int32_t st = kActive;
            double y[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) y[k] = park[k * share + j];
            if (MULTI) S = lds_st[A.st_of_lane[base + j]];
            const HamConst<double> P = ham_const(S.a, y[4], y[7]);
            lane_taken[j] = taken + run_steps<HAM, ZERO_A>(S, P, A.h, A.r_escape, q < left ? q : left, y, st);
            lane_st[j] = st;
#pragma unroll
            for (int k = 0; k < 8; ++k) park[k * share + j] = y[k];
            worked = turn;
        }
        if (m >= 256) {
            j += 256;
            if (j >= m) j -= m;
        }
        __syncthreads();
        // a thread that is ahead may have written a later turn: only where this one goes on, too
        if (look_after(turn) && worked <= turn - kIdleTurns) break;
    }
    for (int32_t i = t; i < m; i += 256) {
        const int32_t taken = lane_taken[i];
        if (taken > 0) {
            A.status[base + i] = lane_st[i];
            A.steps[base + i] += taken;
#pragma unroll
            for (int k = 0; k < 8; ++k) A.state[k * A.n + base + i] = park[k * share + i];
        }
    }
}

// The FP64 step with the invariant monitor folded in every K steps: one thread per
// lane, or the persistent work queue.
template <bool HAM>
__global__ void __launch_bounds__(256) rk4_f64_monitor_kernel(IntArgs A, StTable T, MonArgs MA,
                                                              int32_t multi)
{
    __shared__ Spacetime lds_st[kMaxSt];
    for (int k = threadIdx.x; k < T.n_st; k += blockDim.x) lds_st[k] = T.st[k];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    __shared__ double lds_mon[8 * kMonLanes];
    MonProg<F64Prog<HAM>, HAM> P{F64Prog<HAM>{A, lds_st, multi != 0, T.n_st}, MA, &lds_mon[threadIdx.x]};
    typename MonProg<F64Prog<HAM>, HAM>::Lane L;
    if (!P.load(i, L)) return;
    while (!P.step(L)) {
    }
    P.store(i, L);
}

template <bool HAM>
__global__ void __launch_bounds__(256) rk4_f64_monitor_persistent_kernel(IntArgs A, StTable T,
                                                                         MonArgs MA, int32_t multi,
                                                                         unsigned long long *counter,
                                                                         int32_t chunk)
{
    __shared__ Spacetime lds_st[kMaxSt];
    for (int k = threadIdx.x; k < T.n_st; k += blockDim.x) lds_st[k] = T.st[k];
    __syncthreads();
    __shared__ double lds_mon[8 * kMonLanes];
    MonProg<F64Prog<HAM>, HAM> P{F64Prog<HAM>{A, lds_st, multi != 0, T.n_st}, MA, &lds_mon[threadIdx.x]};
    persistent_loop(P, A.n, counter, chunk);
}

template <bool HAM>
int launch_monitor(const IntArgs &A, const StTable &T, const MonArgs &MA, bool multi, int block,
                   bool persistent, bool may_decline, int32_t sub, unsigned long long *counter,
                   hipStream_t s)
{
    if (persistent) {
        int grid = 0;
        int rc = persistent_grid((const void *)rk4_f64_monitor_persistent_kernel<HAM>, block, A.n, grid);
        if (rc) return rc;
        if (!(may_decline && queue_is_idle(A.n, grid, block))) {
            hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(1), 0, s, counter);
            MALBEC_LAUNCH_CHECK("zero_u64_kernel");
            hipLaunchKernelGGL((rk4_f64_monitor_persistent_kernel<HAM>), dim3(grid), dim3(block), 0, s,
                               A, T, MA, (int32_t)multi, counter, sub);
            MALBEC_LAUNCH_CHECK("rk4_f64_monitor_persistent_kernel");
            return MALBEC_OK;
        }
    }
    hipLaunchKernelGGL((rk4_f64_monitor_kernel<HAM>), dim3(grid_for(A.n, block)), dim3(block), 0, s,
                       A, T, MA, (int32_t)multi);
    MALBEC_LAUNCH_CHECK("rk4_f64_monitor_kernel");
    return MALBEC_OK;
}

template <bool MULTI, bool HAM, bool UNIT_M, bool ZERO_A>
int launch_plain(const IntArgs &A, const StTable &T, int block, int32_t turns, hipStream_t s)
{
    if (turns > 0) {
        const int32_t share = (int32_t)((A.n + turns - 1) / turns);
        hipLaunchKernelGGL((rk4_f64_turns_kernel<MULTI, HAM, UNIT_M, ZERO_A>), dim3(turns), dim3(256),
                           (size_t)share * kTurnLaneBytes, s, A, T, share, kTurnSteps);
        MALBEC_LAUNCH_CHECK("rk4_f64_turns_kernel");
        return MALBEC_OK;
    }
    hipLaunchKernelGGL((rk4_f64_kernel<MULTI, false, HAM, UNIT_M, ZERO_A>), dim3(grid_for(A.n, block)),
                       dim3(block), 0, s, A, T);
    MALBEC_LAUNCH_CHECK("rk4_f64_kernel");
    return MALBEC_OK;
}

// turns: the blocks of a launch in turns, 0 for one thread per lane.
template <bool MULTI, bool CKPT, bool HAM>
int launch_kernel(const IntArgs &A, const StTable &T, int block, int32_t turns, hipStream_t s)
{
    if constexpr (MULTI && !CKPT) return launch_plain<true, HAM, false, false>(A, T, block, turns, s);
    if constexpr (!MULTI && !CKPT) {
        const bool unit = T.st[0].M == 1.0, zero = T.st[0].a == 0.0;
        if (zero) return unit ? launch_plain<false, HAM, true, true>(A, T, block, turns, s)
                              : launch_plain<false, HAM, false, true>(A, T, block, turns, s);
        return unit ? launch_plain<false, HAM, true, false>(A, T, block, turns, s)
                    : launch_plain<false, HAM, false, false>(A, T, block, turns, s);
    }
    hipLaunchKernelGGL((rk4_f64_kernel<MULTI, CKPT, HAM>), dim3(grid_for(A.n, block)), dim3(block), 0, s,
                       A, T);
    MALBEC_LAUNCH_CHECK("rk4_f64_kernel");
    return MALBEC_OK;
}

}  // namespace

int launch_integrate_f64(const malbec_run &run, const StTable &T, const int32_t *st_of_lane,
                         int64_t n, double *state, int32_t *status, int32_t *steps,
                         double *checkpoints, void *ws, hipStream_t s)
{
    const int block = run.block > 0 ? run.block : 256;
    if (block > 256) return fail(MALBEC_EINVAL, "block %d exceeds the kernel's launch bound 256", block);
    const bool multi = st_of_lane != nullptr && T.n_st > 1;
    const bool ham = run.formulation == MALBEC_FORM_HAMILTONIAN;
    if (ham && checkpoints && run.checkpoint_every > 0)
        return fail(MALBEC_ENOTSUP, "checkpoints need the Christoffel formulation");
    const int64_t total = run.n_steps;
    const int64_t chunk = run.steps_per_chunk > 0 ? run.steps_per_chunk : total;
    IntArgs A;
    A.n = n;
    A.state = state;
    A.status = status;
    A.steps = steps;
    A.st_of_lane = multi ? st_of_lane : nullptr;
    A.ckpt = run.checkpoint_every > 0 ? checkpoints : nullptr;
    A.h = run.h;
    A.r_escape = run.r_escape;
    A.ck_every = run.checkpoint_every;
    A.ck_last = run.checkpoint_every > 0 ? (int32_t)(total / run.checkpoint_every) : 0;
    if (run.persistent) {
        if (A.ckpt) return fail(MALBEC_ENOTSUP, "checkpoints need the non-persistent kernel");
        // one launch runs all steps; steps_per_chunk is the retire/refill interval
        A.k0 = 0;
        A.n_steps = (int32_t)total;
        const int32_t sub = run.steps_per_chunk > 0 ? run.steps_per_chunk : 64;
        unsigned long long *counter = (unsigned long long *)ws;
        bool declined = run.block == 0 && run.steps_per_chunk == 0;
        int rc;
        if (!ham)
            rc = launch_queue_f64(A, T, multi, block, sub, declined, counter, s);
        else
            rc = multi ? launch_persistent<true, true>(A, T, block, sub, declined, counter, s)
                       : launch_persistent<false, true>(A, T, block, sub, declined, counter, s);
        if (rc || !declined) return rc;
    }
    for (int64_t k0 = 0; k0 < total; k0 += chunk) {
        A.k0 = (int32_t)k0;
        A.n_steps = (int32_t)((total - k0) < chunk ? (total - k0) : chunk);
        int32_t turns = 0, per_cu = 0;
        int rc = MALBEC_OK;
        if (run.block == 0 && !A.ckpt) rc = turns_blocks(n, A.n_steps, turns, per_cu);
        if (rc) return rc;
        if (A.ckpt)
            rc = multi ? launch_kernel<true, true, false>(A, T, block, 0, s)
                       : launch_kernel<false, true, false>(A, T, block, 0, s);
        else if (ham)
            rc = multi ? launch_kernel<true, false, true>(A, T, block, turns, s)
                       : launch_kernel<false, false, true>(A, T, block, turns, s);
        else
            rc = multi ? launch_kernel<true, false, false>(A, T, block, turns, s)
                       : launch_kernel<false, false, false>(A, T, block, turns, s);
        if (rc) return rc;
    }
    return MALBEC_OK;
}

int launch_monitor_f64(const malbec_run &run, const StTable &T, const int32_t *st_of_lane,
                       int64_t n, double *state, int32_t *status, int32_t *steps, int32_t every,
                       int32_t reset, double *mon, void *ws, hipStream_t s)
{
    const int block = run.block > 0 ? run.block : 256;
    if (block > 256) return fail(MALBEC_EINVAL, "block %d exceeds the kernel's launch bound 256", block);
    const bool multi = st_of_lane != nullptr && T.n_st > 1;
    const bool ham = run.formulation == MALBEC_FORM_HAMILTONIAN;
    const int64_t total = run.n_steps;
    IntArgs A;
    A.n = n;
    A.state = state;
    A.status = status;
    A.steps = steps;
    A.st_of_lane = multi ? st_of_lane : nullptr;
    A.ckpt = nullptr;
    A.h = run.h;
    A.r_escape = run.r_escape;
    A.ck_every = 0;
    A.ck_last = 0;
    A.k0 = 0;
    MonArgs MA{mon, steps, n, every, reset};
    unsigned long long *counter = (unsigned long long *)ws;
    if (run.persistent) {
        A.n_steps = (int32_t)total;
        const int32_t sub = run.steps_per_chunk > 0 ? run.steps_per_chunk : 64;
        const bool may_decline = run.block == 0 && run.steps_per_chunk == 0;
        return ham ? launch_monitor<true>(A, T, MA, multi, block, true, may_decline, sub, counter, s)
                   : launch_monitor<false>(A, T, MA, multi, block, true, may_decline, sub, counter, s);
    }
    const int64_t chunk = run.steps_per_chunk > 0 ? run.steps_per_chunk : total;
    for (int64_t k0 = 0; k0 < total; k0 += chunk) {
        A.k0 = (int32_t)k0;
        A.n_steps = (int32_t)((total - k0) < chunk ? (total - k0) : chunk);
        MA.reset = (k0 == 0) ? reset : 0;
        int rc = ham ? launch_monitor<true>(A, T, MA, multi, block, false, false, 0, counter, s)
                     : launch_monitor<false>(A, T, MA, multi, block, false, false, 0, counter, s);
        if (rc) return rc;
    }
    return MALBEC_OK;
}

}  // namespace malbec
