// Interpolation weights of the gridded metric.  Compiled for the host by the tests.
#pragma once

#include "kerr_accel.hpp"

namespace malbec {

// Lagrange basis on the nodes -1, 0, 1, 2 at u, and six times its derivative:
//   w = {-u (u-1)(u-2)/6, (u+1)(u-1)(u-2)/2, -(u+1) u (u-2)/2, (u+1) u (u-1)/6}.
// One inner weight of each set is formed as what the other three leave of the sum (1 and 0), since the
// rounding of the sum is what the large node values (gamma_thth ~ r^2) carry into the derivatives; the
// sixth goes into the grid's scale, which keeps the constants whole.  With 1/3 and 1/6 for constants the
// rounding of the sum has a preferred sign: the derivative of r^2 on cells of 0.075 is then off by 3.7e-15 in
// the mean and 9.7e-15 rms (relative, over r in [5, 50]), in this form by 7e-19 and 3.4e-15 (with every
// weight from its own product by 8e-18 and 1.1e-14).  After 400 steps on the 801 x 401 Kerr grid, against the
// same interpolant in extended precision: p_r 1.65e-14 -> 2.4e-15 rms (relative), p_theta 1.18e-14 -> 1.3e-15.
// The same time (262,144 lanes x 400 steps 5.83 and 5.85 ms); with one operation fewer, from u^2 and the
// constants 3, 6 and 9, it is 2 % longer, for the constants cost registers.
MALBEC_HD inline void lagrange4(double u, double w[4], double dw6[4])
{
    const double p = fma(u, u, -u);    // u (u - 1)
    const double q = p - 2.0;          // (u + 1)(u - 2)
    w[0] = p * fma(u, -1.0 / 6.0, 1.0 / 3.0);
    w[2] = q * (-0.5 * u);
    w[3] = p * fma(u, 1.0 / 6.0, 1.0 / 6.0);
    w[1] = (1.0 - w[2]) - (w[0] + w[3]);
    const double v = 3.0 * u, t = v * u, e = fma(v, 2.0, -2.0);  // 3 u^2, 6 u - 2
    dw6[0] = e - t;
    dw6[2] = fma(t, -3.0, e + 8.0);
    dw6[3] = t - 1.0;
    dw6[1] = -(dw6[0] + dw6[3]) - dw6[2];
}

}  // namespace malbec
