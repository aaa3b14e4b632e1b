// Geodesics in a numerical metric given in 3+1 form on an (r, theta) grid.
//
// Section 2 writes the line element in 3+1 form (eq. ADM: lapse alpha, shift
// beta^i, spatial metric gamma_ij), gives them for Kerr, and names the 3+1 form as
// the route to numerically computed metrics.  Here a stationary, axisymmetric metric
// with beta = (0, 0, beta^phi) and diagonal gamma is five functions of (r, theta),
//   F = (alpha, beta^phi, gamma_rr, gamma_thth, gamma_phph / sin^2 theta),
// sampled on a uniform grid (node (i, j) holds its five values contiguously: 40 B as
// doubles, 20 B as floats; the values are widened to FP64 on load).
// At a point the kernel takes the tensor product of 4-point Lagrange interpolants
// (16 nodes: four rows of four consecutive nodes, 160 contiguous bytes each), the
// derivatives of that interpolant, the inverse metric
//   g^tt = -1/alpha^2, g^tphi = beta^phi/alpha^2,
//   g^phph = 1/gamma_phph - (beta^phi)^2/alpha^2, g^rr = 1/gamma_rr, g^thth = 1/gamma_thth
// and Hamilton's equations (eq. Ham) on (x^mu, p_mu) with classic RK4 (p_t and p_phi are
// constants).
//
// What bounds it: FP64 VALU issue, 378 instructions per right-hand side (220 of them the
// interpolation's fma), at two waves per SIMD, the most that a 640 B stencil per lane
// allows (Stencil below).  Measured on one MI355X, the same machine before (stencil
// entirely in LDS, one wave per SIMD with double nodes; derivatives of the inverse
// metric; four inlined copies of the right-hand side) and after:
//   801 x 401 grid, double nodes, 262,144 lanes x 400 steps: 10.92 -> 5.85 ms
//     (1.79 x 10^10 lane-steps/s; VALU active 0.52 -> 0.77, 2006 -> 1520 per step)
//   401 x 201 grid, float nodes, 100,003 lanes x 500 steps: 5.00 -> 3.5 ms
// Cell changes cost 15 % of it (1.42 against 1.66 ms on 131,072 lanes x 200 steps that
// stay in their cells or not).  Gathering for the few lanes that change cell by the whole
// wavefront (one load per such lane instead of 40 under its mask) was 4 % slower: the
// exchange through LDS lengthens the wait.
#include "grid_weights.hpp"
#include "internal.hpp"
#include "turns.hpp"

namespace malbec {

namespace {

struct GridArgs {
    int64_t n;
    double *state;
    int32_t *status;
    int32_t *steps;
    const void *nodes;  // Node[nr * nth * 5], Node = double or float
    int32_t nr, nth;
    double r0, idr, th0, idth;   // inverse spacings
    double idr6, idth6;          // a sixth of them
    double rlo, rhi, tlo, thi;   // interior (stencils and stage points stay inside)
    double r_stop, r_escape, h;
    int32_t n_steps;
};

// x truncated to an integer for every double: the instruction saturates and takes a NaN to 0, where
// the language leaves such conversions undefined.
__device__ __forceinline__ int32_t truncated(double x)
{
    int32_t i;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(x));
    return i;
}

// Cell index of x on a grid of n nodes (the stencil starts one node before) and the
// offset u in it.  The index is clamped to [1, n - 3] as an integer, so every access stays
// inside the grid, also for stage points off the grid and for NaN.
__device__ __forceinline__ int32_t cell(double x, double x0, double ih, int32_t n, double &u)
{
    const double q = (x - x0) * ih;
    const int32_t i = min(max(truncated(q), 1), n - 3);
    u = q - (double)i;
    return i;
}

// Stencil of one lane: the 16 nodes x 5 values of the cell that the lane is in, widened
// to FP64 when it is gathered, with two of the four rows in registers and two in LDS.
// The four stage points of a step, and the next steps, mostly lie in the same cell (a
// stage moves a few thousandths in r and theta against cells of 0.075 and 0.0075 on the
// benchmark grid), so the grid itself is read only when a lane changes cell.  Half of
// the stencil in LDS is 320 B per lane: 512 lanes fill a CU's 160 KB, two waves per
// SIMD, which the 80 registers of the other half also allow.  (All of it in LDS, 640 B
// per lane, leaves one wave per SIMD and makes the LDS reads, 40 of 16 B per lane and
// right-hand side, as long as the arithmetic.)  A row's 20 values (value k of node b at
// e = b * 5 + k) are contiguous in the grid but aligned to one value only; they are
// gathered, held and read as the ten pairs they come in.  Each wavefront has its own
// part of the LDS, chunk m of its lane l at [m * 64 + l]: conflict-free, at offsets that
// do not depend on the block size.
typedef double Double2 __attribute__((ext_vector_type(2)));
template <typename Node>
struct Row {
    typedef Node Pair __attribute__((ext_vector_type(2), aligned(sizeof(Node))));
};
constexpr int kLdsChunks = 20;  // third and fourth row
struct Stencil {
    Double2 *lds;        // this lane's column of its wavefront's part
    int32_t ci, cj;      // cell held (-1: none)
    Double2 row[2][10];  // first and second row
};

template <typename Node>
__device__ __forceinline__ void stencil_load(const GridArgs &A, int32_t i, int32_t j, Stencil &C)
{
    typedef typename Row<Node>::Pair Pair;
    const int64_t pitch = (int64_t)A.nth * 5;
    const Node *p = (const Node *)A.nodes + (int64_t)(i - 1) * pitch + (int64_t)(j - 1) * 5;
    Pair g[2][10];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int e = 0; e < 10; ++e) g[a][e] = *(const Pair *)(p + (2 + a) * pitch + 2 * e);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int e = 0; e < 10; ++e) {
            const Pair q = *(const Pair *)(p + a * pitch + 2 * e);
            C.row[a][e] = Double2{(double)q[0], (double)q[1]};
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int e = 0; e < 10; ++e)
            C.lds[(a * 10 + e) * 64] = Double2{(double)g[a][e][0], (double)g[a][e][1]};
    }
    C.ci = i;
    C.cj = j;
    __builtin_amdgcn_sched_barrier(0);
}

// F, 6 dF/du_r and 6 dF/du_theta (u: the offset in cells) of the five functions at
// (r, theta).  Function by function: the theta contraction of its four rows, value and
// derivative, then the r contraction (44 fma).
template <typename Node>
__device__ __forceinline__ void grid_eval(const GridArgs &A, double r, double th, double F[5],
                                          double Fr[5], double Ft[5], Stencil &C)
{
    double ur, ut, wr[4], dwr[4], wt[4], dwt[4];
    const int32_t i = cell(r, A.r0, A.idr, A.nr, ur);
    const int32_t j = cell(th, A.th0, A.idth, A.nth, ut);
    if (i != C.ci || j != C.cj) stencil_load<Node>(A, i, j, C);
    lagrange4(ur, wr, dwr);
    lagrange4(ut, wt, dwt);
    __builtin_amdgcn_sched_barrier(0);
    Double2 q[4][10];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int e = 0; e < 10; ++e) {
            q[a][e] = C.row[a][e];
            q[2 + a][e] = C.lds[(a * 10 + e) * 64];
        }
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        double f[4][4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
#pragma unroll
            for (int b = 0; b < 4; ++b) f[a][b] = q[a][(b * 5 + k) / 2][(b * 5 + k) % 2];
        }
        F[k] = Fr[k] = Ft[k] = 0.0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const double v = fma(wt[3], f[a][3], fma(wt[2], f[a][2], fma(wt[1], f[a][1], wt[0] * f[a][0])));
            const double vt = fma(dwt[3], f[a][3], fma(dwt[2], f[a][2], fma(dwt[1], f[a][1], dwt[0] * f[a][0])));
            F[k] = fma(wr[a], v, F[k]);
            Fr[k] = fma(dwr[a], v, Fr[k]);
            Ft[k] = fma(wr[a], vt, Ft[k]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

__device__ __forceinline__ bool inside(const GridArgs &A, double r, double th)
{
    return r >= A.rlo && r <= A.rhi && th >= A.tlo && th <= A.thi;
}

// Canonical right-hand side with the gridded metric.  With
// u^a = g^ab p_b, dp_l/dtau = -(1/2) d_l g^ab p_a p_b = (1/2) d_l g_ab u^a u^b, which in
// 3+1 form, with w = u^phi + beta^phi u^t = p_phi / gamma_phph, is
//   -alpha d_l alpha (u^t)^2 + p_phi u^t d_l beta^phi
//     + (1/2) [d_l gamma_rr (u^r)^2 + d_l gamma_thth (u^theta)^2 + d_l gamma_phph w^2]:
// no derivative of the inverse metric is formed.  One reciprocal of the product of
// alpha^2 and the three gammas gives all four inverses.
template <typename Node>
__device__ __forceinline__ void grid_ham(const GridArgs &A, const HamConst<double> &P, Stencil &C,
                                         const TrigBase<false> &trig, double r, double th, double pr,
                                         double pth, double &dt, double &dr, double &dth,
                                         double &dph, double &dpr, double &dpth)
{
    double F[5], Fr[5], Ft[5];
    grid_eval<Node>(A, r, th, F, Fr, Ft, C);
    double s, c;
    trig.at(th, s, c);
    const double s2 = s * s, sc = s * c;
    const double al = F[0], be = F[1];
    const double al2 = al * al, gpp = F[4] * s2;
    const double p12 = al2 * F[2], p34 = F[3] * gpp;
    const double inv = recip(p12 * p34);
    const double i12 = inv * p34, i34 = inv * p12;
    dt = (i12 * F[2]) * fma(be, P.pph, -P.pt);
    const double w = (i34 * F[3]) * P.pph;
    dph = fma(-be, dt, w);
    dr = (i12 * al2) * pr;
    dth = (i34 * gpp) * pth;
    const double c0 = -al * (dt * dt), c1 = P.pph * dt;
    const double w2 = w * w, w2s2 = w2 * s2, rr = dr * dr, hh = dth * dth;
    auto force = [&](const double D[5]) {
        const double kin = fma(rr, D[2], fma(hh, D[3], w2s2 * D[4]));
        return fma(0.5, kin, fma(c0, D[0], c1 * D[1]));
    };
    dpr = A.idr6 * force(Fr);
    dpth = fma(A.idth6, force(Ft), (w2 * sc) * F[4]);
}

// Up to n_steps steps of an active lane from y, which receives its state after them; returns
// the steps evaluated and sets st.
template <typename Node>
__device__ __forceinline__ int32_t grid_steps(const GridArgs &A, const HamConst<double> &P, Stencil &C,
                                              int32_t n_steps, double y[8], int32_t &st)
{
    int32_t taken = 0;
    const double hh = 0.5 * A.h, h6 = A.h * (1.0 / 6.0);
    while (taken < n_steps) {
        // One RK4 step, its stages in a loop: one copy of the right-hand side, so that the
        // stencil's registers have one place each.  The stop rules at the stage points: the
        // first that is in the stop zone or off the grid decides.
        TrigBase<false> trig;
        trig.set(y[2]);
        double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        double r = y[1], th = y[2], pr = y[5], pth = y[6];
        int32_t out = kActive;
#pragma unroll 1
        for (int stage = 0; stage < 4; ++stage) {
            const bool good = (r > A.r_stop) & (r <= A.rhi) & (th >= A.tlo) & (th <= A.thi);
            if (!good && stage > 0 && out == kActive) out = r <= A.r_stop ? kHorizon : kNonfinite;
            double dt, dr, dth, dph, dpr, dpth;
            grid_ham<Node>(A, P, C, trig, r, th, pr, pth, dt, dr, dth, dph, dpr, dpth);
            const double b = stage == 0 || stage == 3 ? 1.0 : 2.0;  // weights 1, 2, 2, 1
            acc[0] = fma(b, dt, acc[0]);
            acc[1] = fma(b, dr, acc[1]);
            acc[2] = fma(b, dth, acc[2]);
            acc[3] = fma(b, dph, acc[3]);
            acc[4] = fma(b, dpr, acc[4]);
            acc[5] = fma(b, dpth, acc[5]);
            const double a = stage == 2 ? A.h : hh;  // offset of the next stage point
            r = fma(a, dr, y[1]);
            th = fma(a, dth, y[2]);
            pr = fma(a, dpr, y[5]);
            pth = fma(a, dpth, y[6]);
        }
        ++taken;
        const double y1[8] = {fma(h6, acc[0], y[0]), fma(h6, acc[1], y[1]), fma(h6, acc[2], y[2]),
                              fma(h6, acc[3], y[3]), y[4], fma(h6, acc[4], y[5]),
                              fma(h6, acc[5], y[6]), y[7]};
        // the common outcome first (r_stop and r_escape lie inside the grid and its theta
        // range inside (0, pi); an infinite or NaN p_t or p_phi makes t or phi so)
        const bool go = (out == kActive) & (y1[1] > A.r_stop) & (y1[1] < A.r_escape) &
                        (y1[2] >= A.tlo) & (y1[2] <= A.thi) & (bool)__builtin_isfinite(y1[0]) &
                        (bool)__builtin_isfinite(y1[3]) & (bool)__builtin_isfinite(y1[5]) &
                        (bool)__builtin_isfinite(y1[6]);
        if (!go) {
            if (out == kActive && (!usable(y1) || !inside(A, y1[1], y1[2]))) out = kNonfinite;
            if (out != kActive) {
                st = out;
                break;
            }
            if (y1[1] <= A.r_stop) st = kHorizon;
            else if (y1[1] >= A.r_escape) st = kEscape;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) y[c] = y1[c];
        if (st != kActive) break;
    }
    return taken;
}

// At most 256 registers, the two waves per SIMD that the stencils' LDS allows; four (16 in turns) that
// live across the loop are spilled, 20 B (52 B) per lane.
template <typename Node>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
rk4_grid_kernel(GridArgs A)
{
    extern __shared__ Double2 lds_stencil[];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    int32_t st = A.status[i];
    if (st != kActive) return;
    double y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) y[k] = A.state[k * A.n + i];
    const HamConst<double> P{y[4], y[7], 0.0, 0.0};
    Stencil C;
    C.lds = &lds_stencil[(threadIdx.x / 64u) * (kLdsChunks * 64) + threadIdx.x % 64u];
    C.ci = C.cj = -1;
    const int32_t taken = grid_steps<Node>(A, P, C, A.n_steps, y, st);
    const int64_t ie = opaque(i);
#pragma unroll
    for (int k = 0; k < 8; ++k) A.state[k * A.n + ie] = y[k];
    A.status[ie] = st;
    A.steps[ie] += taken;
}

// A batch that fills the chip unevenly, in turns (rk4_f64_turns_kernel in integrate.hip).  The stencils
// take the LDS, so the lanes that wait are parked where they came from, in the state arrays (L2).
template <typename Node>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
rk4_grid_turns_kernel(GridArgs A, int32_t share, int32_t q)
{
    extern __shared__ Double2 lds_stencil[];
    const int64_t base = (int64_t)blockIdx.x * share;
    const int64_t rest = A.n - base;
    const int32_t m = rest < share ? (int32_t)rest : share;  // lanes of this block (may be <= 0)
    const int32_t turns = turns_of_block(A.n_steps, q, m);
    Stencil C;
    C.lds = &lds_stencil[(threadIdx.x / 64u) * (kLdsChunks * 64) + threadIdx.x % 64u];
    bool worked = false;  // a lane of this thread stepped since the last look
    int32_t j = (int32_t)threadIdx.x, had = 0;  // the lane, and the turns it has had
    for (int32_t turn = 0; turn < turns; ++turn) {
        const int32_t steps = steps_of_turn(A.n_steps, q, had);
        if (j < m && steps > 0) {
            const int64_t i = base + j;
            int32_t st = A.status[i];
            if (st == kActive) {
                worked = true;
                double y[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) y[k] = A.state[k * A.n + i];
                const HamConst<double> P{y[4], y[7], 0.0, 0.0};
                C.ci = C.cj = -1;
                const int32_t taken = grid_steps<Node>(A, P, C, steps, y, st);
                const int64_t ie = opaque(i);
#pragma unroll
                for (int k = 0; k < 8; ++k) A.state[k * A.n + ie] = y[k];
                A.status[ie] = st;
                A.steps[ie] += taken;
            }
        }
        next_turn(m, j, had);
        __syncthreads();
        if (look_after(turn)) {
            // the threads' answers go through the stencils' LDS (free between turns; another word of LDS
            // would leave room for one block per CU instead of two)
            if (threadIdx.x == 0) lds_stencil[0][0] = 0.0;
            __syncthreads();
            if (worked) lds_stencil[0][0] = 1.0;
            __syncthreads();
            const bool any = lds_stencil[0][0] != 0.0;
            __syncthreads();
            if (!any) break;
            worked = false;
        }
    }
}

// Kerr's 3+1 functions (Section 2) at every node, computed in FP64 and stored as Node.
template <typename Node>
__global__ void __launch_bounds__(256) grid_fill_kerr_kernel(Node *nodes, int32_t nr, int32_t nth,
                                                             double r0, double dr, double th0,
                                                             double dth, double M, double a)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= (int64_t)nr * nth) return;
    const int64_t i = p / nth, j = p % nth;
    const double r = r0 + (double)i * dr, th = th0 + (double)j * dth;
    double s, c;
    sincos(th, &s, &c);
    const double r2a2 = r * r + a * a;
    const double rho2 = r * r + a * a * c * c;
    const double Delta = r * r - 2.0 * M * r + a * a;
    const double Sigma = r2a2 * r2a2 - a * a * Delta * s * s;
    Node *F = nodes + p * 5;
    F[0] = (Node)sqrt(rho2 * Delta / Sigma);
    F[1] = (Node)(-2.0 * M * a * r / Sigma);
    F[2] = (Node)(rho2 / Delta);
    F[3] = (Node)rho2;
    F[4] = (Node)(Sigma / rho2);
}

}  // namespace

int launch_grid_fill_kerr(const malbec_grid &g, double M, double a, void *nodes, hipStream_t s)
{
    const int block = 256;
    const int64_t np = (int64_t)g.nr * g.nth;
    if (g.node_precision == MALBEC_GRID_F32)
        hipLaunchKernelGGL(grid_fill_kerr_kernel<float>, dim3(grid_for(np, block)), dim3(block), 0, s,
                           (float *)nodes, g.nr, g.nth, g.r0, g.dr, g.th0, g.dth, M, a);
    else
        hipLaunchKernelGGL(grid_fill_kerr_kernel<double>, dim3(grid_for(np, block)), dim3(block), 0,
                           s, (double *)nodes, g.nr, g.nth, g.r0, g.dr, g.th0, g.dth, M, a);
    MALBEC_LAUNCH_CHECK("grid_fill_kerr_kernel");
    return MALBEC_OK;
}

// The blocks of a launch in turns, 0 where one thread per lane is the better launch.  With
// n / (256 lanes per CU) = w + f, w whole, min(w, 2) blocks per CU (their stencils fill its LDS).  A turn
// gathers every lane's stencil again, so it is worth less here than where lanes park in LDS.  One
// thread per lane and in turns on one MI355X, ms (400 steps, 801 x 401 double and 401 x 201 float nodes;
// 100 steps, double nodes):
//   w + f   1.05          1.3           1.5           2.05          2.5           3.05          3.5
//         2.87 2.26     2.93 2.77     2.96 3.18     4.67 3.66     4.63 4.34     6.04 5.32     6.06 6.03
//         2.76 1.99     2.77 2.43     2.79 2.78     4.22 3.31     4.27 3.87     5.70 4.84     5.60 5.43
//         0.76 0.66     0.77 0.78     0.77 0.87     1.14 0.99     1.15 1.13     1.47 1.39     1.48 1.57
// Turns of 32 steps, of 16 below 160 (at 400 steps 16 is 3-5 % slower, at 100 32 is 5 % slower).
static int grid_turns(int64_t n, int32_t n_steps, int32_t &blocks)
{
    blocks = 0;
    if (n_steps < 100) return MALBEC_OK;
    int dev = 0, n_cu = 0;
    MALBEC_HIP_CHECK(hipGetDevice(&dev));
    MALBEC_HIP_CHECK(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    const int64_t level = (int64_t)n_cu * 256, w = n / level;
    const double f = (double)(n - w * level) / (double)level;
    const double most = w == 1 ? 0.25 : w == 2 ? 0.5 : w == 3 ? 0.3 : 0.0;
    if (f > 0.0 && f <= most) blocks = (int32_t)(w < 2 ? n_cu : 2 * n_cu);
    return MALBEC_OK;
}

int launch_integrate_grid(const malbec_run &run, const malbec_grid &g, int64_t n, double *state,
                          int32_t *status, int32_t *steps, hipStream_t s)
{
    // A batch that leaves CUs idle is spread in blocks of one wavefront, each with the LDS and
    // L1 of a CU to itself: 10,000 lanes x 100 steps take 454 us in blocks of 64 and 508 us in
    // blocks of 256; at 30,000 lanes they are level (498 and 520 us), and from 65,536 lanes
    // on blocks of 256 are ahead (583 against 597 us, 6.0 against 6.2 ms at 1,048,576).
    const int block = run.block > 0 ? run.block : n <= 32768 ? 64 : 256;
    if (block > 256) return fail(MALBEC_EINVAL, "block %d exceeds the kernel's launch bound 256", block);
    GridArgs A;
    A.n = n;
    A.state = state;
    A.status = status;
    A.steps = steps;
    A.nodes = g.nodes;
    A.nr = g.nr;
    A.nth = g.nth;
    A.r0 = g.r0;
    A.idr = 1.0 / g.dr;
    A.th0 = g.th0;
    A.idth = 1.0 / g.dth;
    A.idr6 = (double)(1.0L / (6.0L * g.dr));
    A.idth6 = (double)(1.0L / (6.0L * g.dth));
    A.rlo = g.r0 + g.dr;
    A.rhi = g.r0 + (double)(g.nr - 2) * g.dr;
    A.tlo = g.th0 + g.dth;
    A.thi = g.th0 + (double)(g.nth - 2) * g.dth;
    A.r_stop = g.r_stop;
    A.r_escape = run.r_escape;
    A.h = run.h;
    const size_t lds = (size_t)block * kLdsChunks * sizeof(Double2);
    const int64_t total = run.n_steps;
    const int64_t chunk = run.steps_per_chunk > 0 ? run.steps_per_chunk : total;
    for (int64_t k0 = 0; k0 < total; k0 += chunk) {
        A.n_steps = (int32_t)((total - k0) < chunk ? (total - k0) : chunk);
        int32_t turns = 0;
        if (run.block == 0) {
            const int rc = grid_turns(n, A.n_steps, turns);
            if (rc) return rc;
        }
        if (turns > 0) {
            const int32_t share = (int32_t)((n + turns - 1) / turns);
            const int32_t q = A.n_steps < 160 ? 16 : 32;
            if (g.node_precision == MALBEC_GRID_F32)
                hipLaunchKernelGGL(rk4_grid_turns_kernel<float>, dim3(turns), dim3(256), lds, s, A, share, q);
            else
                hipLaunchKernelGGL(rk4_grid_turns_kernel<double>, dim3(turns), dim3(256), lds, s, A, share, q);
            MALBEC_LAUNCH_CHECK("rk4_grid_turns_kernel");
            continue;
        }
        if (g.node_precision == MALBEC_GRID_F32)
            hipLaunchKernelGGL(rk4_grid_kernel<float>, dim3(grid_for(n, block)), dim3(block), lds, s, A);
        else
            hipLaunchKernelGGL(rk4_grid_kernel<double>, dim3(grid_for(n, block)), dim3(block), lds, s, A);
        MALBEC_LAUNCH_CHECK("rk4_grid_kernel");
    }
    return MALBEC_OK;
}

}  // namespace malbec
