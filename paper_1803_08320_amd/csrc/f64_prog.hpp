// What the FP64 fixed-step kernels share: their arguments, the step of either formulation, the
// loop over steps, and a lane as a work item of the persistent queue.
#pragma once

#include "internal.hpp"
#include "persistent.hpp"

namespace malbec {

struct IntArgs {
    int64_t n;
    double *state;
    int32_t *status;
    int32_t *steps;
    const int32_t *st_of_lane;
    double *ckpt;      // checkpoint slots or nullptr
    double h;
    double r_escape;
    int32_t n_steps;   // steps in this launch
    int32_t k0;        // index of this launch's first step within the call
    int32_t ck_every;  // K (0 = none)
    int32_t ck_last;   // index of the last slot of the call
};

namespace {

__device__ __forceinline__ void copy8(double dst[8], const double src[8])
{
#pragma unroll
    for (int c = 0; c < 8; ++c) dst[c] = src[c];
}

// One FP64 RK4 step of either formulation: the Christoffel form on (x, u), or
// Hamilton's equations on (x, p) with the lane's constants p_t, p_phi in P.
template <bool HAM, bool ZERO_A = false>
__device__ __forceinline__ void step_f64(const Spacetime &S, const HamConst<double> &P, double h,
                                         const double y[8], double y1[8], double sr[3])
{
    if (HAM)
        rk4_step_ham_f64<ZERO_A>(S, P, h, y, y1, sr);
    else
        rk4_step_f64<true, TabGlobal, ZERO_A>(S, h, y, y1, sr);
}

// Up to n >= 1 steps of an active lane from y, which receives its state after them; returns
// the steps evaluated and sets st.  Two steps per iteration, the second with the roles of
// y and y1 swapped, so that an accepted step never copies the state.  The common outcome
// of the stop rules is tested first.
template <bool HAM, bool ZERO_A = false>
__device__ __forceinline__ int32_t run_steps(const Spacetime &S, const HamConst<double> &P, double h,
                                             double r_escape, int32_t n, double y[8], int32_t &st)
{
    double y1[8];
    int32_t ks = 0;
    for (;;) {
        double sr[3];
        bool accept = true;
        step_f64<HAM, ZERO_A>(S, P, h, y, y1, sr);
        ++ks;
        if (!still_active_f64(S, r_escape, sr, y1)) st = terminate_f64(S, r_escape, sr, y1, accept);
        if (st != kActive || ks == n) {
            if (accept) copy8(y, y1);
            return ks;
        }
        step_f64<HAM, ZERO_A>(S, P, h, y1, y, sr);
        ++ks;
        accept = true;
        if (!still_active_f64(S, r_escape, sr, y)) st = terminate_f64(S, r_escape, sr, y, accept);
        if (st != kActive || ks == n) {
            if (!accept) copy8(y, y1);
            return ks;
        }
    }
}

// One lane of the batch as a work item of the persistent driver; the step is the
// same rk4_step_f64 / terminate_f64 sequence as the one-thread-per-lane kernel.
template <bool HAM>
struct F64Prog {
    const IntArgs &A;
    const Spacetime *table;  // LDS copy (mixed batch) or kernel argument
    bool multi;
    int32_t n_st;
    struct Lane {
        double y[8];
        Spacetime S;
        HamConst<double> P;
        int32_t st, taken;
    };
    // Read again from the kernel's arguments in the Hamiltonian form alone, whose persistent
    // kernel is 2 % faster with it (the Christoffel form's is not).
    __device__ __forceinline__ auto args() const
    {
        if constexpr (HAM)
            return first_arg<IntArgs>();
        else
            return &A;
    }
    __device__ __forceinline__ bool load(int64_t i, Lane &L)
    {
        const auto *A = args();
        L.st = A->status[i];
        if (L.st != kActive) return false;
        int32_t sid = 0;
        if (multi) {
            sid = A->st_of_lane[i];
            if (sid < 0 || sid >= n_st) {
                A->status[i] = kNonfinite;
                return false;
            }
        }
        L.S = table[sid];
#pragma unroll
        for (int k = 0; k < 8; ++k) L.y[k] = A->state[k * A->n + i];
        L.P = ham_const(L.S.a, L.y[4], L.y[7]);
        L.taken = 0;
        return A->n_steps > 0;
    }
    __device__ __forceinline__ bool step(Lane &L)
    {
        double y1[8], sr[3];
        step_f64<HAM>(L.S, L.P, A.h, L.y, y1, sr);
        ++L.taken;
        bool accept = true;  // the common outcome of the stop rules first, as rk4_f64_kernel
        if (!still_active_f64(L.S, A.r_escape, sr, y1)) L.st = terminate_f64(L.S, A.r_escape, sr, y1, accept);
        if (accept) copy8(L.y, y1);
        return L.st != kActive || L.taken == A.n_steps;
    }
    __device__ __forceinline__ void store(int64_t item, const Lane &L)
    {
        const auto *A = args();
        const int64_t i = opaque(item);
#pragma unroll
        for (int k = 0; k < 8; ++k) A->state[k * A->n + i] = L.y[k];
        A->status[i] = L.st;
        A->steps[i] += L.taken;
    }
    __device__ static __forceinline__ void state64(const Lane &L, double y[8]) { copy8(y, L.y); }
};

template <bool MULTI, bool HAM>
__global__ void __launch_bounds__(256) rk4_f64_persistent_kernel(IntArgs A, StTable T,
                                                                 unsigned long long *counter,
                                                                 int32_t chunk)
{
    __shared__ Spacetime lds_st[kMaxSt];
    for (int k = threadIdx.x; k < T.n_st; k += blockDim.x) lds_st[k] = T.st[k];
    __syncthreads();
    F64Prog<HAM> P{A, lds_st, MULTI, T.n_st};
    persistent_loop(P, A.n, counter, chunk);
}

template <bool MULTI, bool HAM>
int launch_persistent(const IntArgs &A, const StTable &T, int block, int32_t sub, bool &declined,
                      unsigned long long *counter, hipStream_t s)
{
    int grid = 0;
    int rc = persistent_grid((const void *)rk4_f64_persistent_kernel<MULTI, HAM>, block, A.n, grid);
    if (rc) return rc;
    declined = declined && queue_is_idle(A.n, grid, block);
    if (declined) return MALBEC_OK;
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(1), 0, s, counter);
    MALBEC_LAUNCH_CHECK("zero_u64_kernel");
    hipLaunchKernelGGL((rk4_f64_persistent_kernel<MULTI, HAM>), dim3(grid), dim3(block), 0, s, A, T,
                       counter, sub);
    MALBEC_LAUNCH_CHECK("rk4_f64_persistent_kernel");
    return MALBEC_OK;
}

}  // namespace

// The persistent kernel of the Christoffel form (queue.hip).  declined: in, whether the launch
// may be left to one thread per lane; out, whether it was.
int launch_queue_f64(const IntArgs &A, const StTable &T, bool multi, int block, int32_t sub,
                     bool &declined, unsigned long long *counter, hipStream_t s);

}  // namespace malbec
