"""The right-hand sides and the RK4 step that the FP64 fixed-step kernels run
(kerr_accel_half, rk4_step_half, kerr_ham_s2), compiled for the host, against the
oracle."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from test_host_rhs import ROOT, _p, sample_states

SRC = r"""
#include "kerr_accel.hpp"
#include "ham_accel.hpp"
struct Half {
    double M, a;
    void operator()(int, double r, double th, double ut, double ur, double uth, double uph,
                    double &at2, double &ar, double &ath, double &aph2) const {
        const double s = std::sin(th), c = std::cos(th);
        malbec::kerr_accel_half<double>(M, a, r, s * s, s * c, ut, ur, uth, uph, at2, ar, ath, aph2);
    }
};
struct HalfVjp : Half {
    double Ys[4][6];
    double &Y(int st, int k) { return Ys[st][k]; }
    void keep() {}
    void prepare(int, double) {}
    void vjp(int, double r, double th, double ut, double ur, double uth, double uph, double bt, double br,
             double bh, double bp, double &rb, double &thb, double ub[4]) const {
        const double s = std::sin(th), c = std::cos(th);
        malbec::kerr_accel_half_vjp<double>(M, a, r, s * s, s * c, ut, ur, uth, uph, bt, br, bh, bp, rb,
                                            thb, ub);
    }
};
extern "C" void half_vjp(double M, double a, const double *y, const double *b, double *g) {
    HalfVjp f{{M, a}, {}};
    f.vjp(0, y[1], y[2], y[4], y[5], y[6], y[7], 2 * b[0], b[1], b[2], 2 * b[3], g[0], g[1], g + 2);
}
extern "C" void full_vjp(double M, double a, const double *y, const double *b, double *g) {
    const double s = std::sin(y[2]), c = std::cos(y[2]);
    double sb, cb;
    malbec::kerr_accel_vjp<double>(M, a, y[1], s, c, y[4], y[5], y[6], y[7], b[0], b[1], b[2], b[3], g[0],
                                   sb, cb, g + 2);
    g[1] = sb * c - cb * s;
}
extern "C" void half_step_vjp(double M, double a, double h, const double *y, double *lam) {
    HalfVjp f{{M, a}, {}};
    malbec::rk4_vjp_half(f, h, y, lam);
}
extern "C" void half_rhs(double M, double a, const double *y, double *f) {
    for (int k = 0; k < 4; ++k) f[k] = y[4 + k];
    Half h{M, a};
    h(0, y[1], y[2], y[4], y[5], y[6], y[7], f[4], f[5], f[6], f[7]);
    f[4] *= 2.0;
    f[7] *= 2.0;
}
extern "C" void half_step(double M, double a, double h, const double *y, double *y1, double *sr) {
    Half f{M, a};
    malbec::rk4_step_half(f, h, y, y1, sr);
}
extern "C" void ham_s2_rhs(double M, double a, const double *z, double *f) {
    const double s = std::sin(z[2]), c = std::cos(z[2]);
    malbec::kerr_ham_s2<double>(M, a, z[1], s * s, s * c, z[5], z[6], malbec::ham_const(a, z[4], z[7]),
                                f[0], f[1], f[2], f[3], f[5], f[6]);
    f[4] = 0.0;
    f[7] = 0.0;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("hostrhs64")
    src, so = d / "host.cpp", d / "libhost.so"
    src.write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
                    "-I", os.path.join(ROOT, "paper_1803_08320_amd", "csrc"), str(src), "-o",
                    str(so)], check=True)
    lib = C.CDLL(str(so))
    dp = C.POINTER(C.c_double)
    lib.half_rhs.argtypes = lib.ham_s2_rhs.argtypes = [C.c_double, C.c_double, dp, dp]
    lib.half_vjp.argtypes = lib.full_vjp.argtypes = [C.c_double, C.c_double, dp, dp, dp]
    lib.half_step_vjp.argtypes = [C.c_double, C.c_double, C.c_double, dp, dp]
    lib.half_step.argtypes = [C.c_double, C.c_double, C.c_double, dp, dp, dp]
    return lib


@pytest.mark.parametrize("M,a", [(1.0, 0.0), (1.0, 0.9), (1.0, 1.0), (2.5, 1.7)])
def test_regrouped_right_hand_sides_match_oracle(orc, host, M, a):
    """To 1e-13 of the largest component (the bound of the forms they regroup)."""
    s0 = sample_states(orc, a / M, 200, 61)
    for i in range(s0.shape[1]):
        y = np.ascontiguousarray(s0[:, i])
        y[1] *= M  # the sampler's unit is M
        y[6:] /= M
        f, ref = np.zeros(8), orc.rhs(M, a, y)
        host.half_rhs(M, a, _p(y), _p(f))
        assert np.max(np.abs(f - ref)) <= 1e-13 * np.max(np.abs(ref))
        z = np.concatenate([y[:4], orc.metric(M, a, y[1], y[2]) @ y[4:]])
        ref = orc.rhs_hamiltonian(M, a, z)
        host.ham_s2_rhs(M, a, _p(z), _p(f))
        assert np.max(np.abs(f - ref)) <= 1e-13 * np.max(np.abs(ref))


@pytest.mark.parametrize("a", [0.0, 0.9])
def test_half_step_matches_oracle(orc, host, a):
    s0 = sample_states(orc, a, 64, 62)
    ref, _, _ = orc.integrate([(1.0, a)], s0, 0.02, 1, r_escape=1e300, horizon_factor=0.0)
    for i in range(s0.shape[1]):
        y, y1, sr = np.ascontiguousarray(s0[:, i]), np.zeros(8), np.zeros(3)
        host.half_step(1.0, a, 0.02, _p(y), _p(y1), _p(sr))
        assert np.max(np.abs(y1 - ref[:, i]) / (np.abs(ref[:, i]) + 1.0)) <= 1e-14
        assert abs(sr[0] - (y[1] + 0.01 * y[5])) <= 1e-14 * y[1]


@pytest.mark.parametrize("M,a", [(1.0, 0.0), (1.0, 0.9), (1.0, 1.0), (2.5, 1.7)])
def test_transposed_jacobians_agree(orc, host, M, a):
    """The transposed Jacobian of the regrouped acceleration against that of the first form,
    to 1e-12 of the sum of the magnitudes it adds up (about 100 roundings, each of terms up
    to a hundred times their sum)."""
    s0 = sample_states(orc, a / M, 100, 63)
    rng = np.random.default_rng(64)
    for i in range(s0.shape[1]):
        y = np.ascontiguousarray(s0[:, i])
        y[1] *= M
        y[6:] /= M
        b, got, want, col = rng.standard_normal(4), np.zeros(6), np.zeros(6), np.zeros(6)
        host.half_vjp(M, a, _p(y), _p(b), _p(got))
        host.full_vjp(M, a, _p(y), _p(b), _p(want))
        scale = np.zeros(6)
        for k in range(4):
            unit = np.zeros(4)
            unit[k] = b[k]
            host.full_vjp(M, a, _p(y), _p(unit), _p(col))
            scale += np.abs(col)
        assert np.all(np.abs(got - want) <= 1e-12 * scale + 1e-300), (i, got, want)


@pytest.mark.parametrize("a", [0.0, 0.9])
def test_half_step_vjp_is_the_transpose_of_the_oracle_tangent(orc, host, a):
    """<lam, J v> = <J^T lam, v>, to the bound of the first form's test."""
    s0 = sample_states(orc, a, 64, 57)
    rng = np.random.default_rng(58)
    for i in range(s0.shape[1]):
        y = np.ascontiguousarray(s0[:, i])
        v, lam = rng.standard_normal(8), rng.standard_normal(8)
        _, jv = orc.tangent(1.0, a, 0.02, 1, y, v)
        jt = lam.copy()
        host.half_step_vjp(1.0, a, 0.02, _p(y), _p(jt))
        scale = np.abs(lam) @ np.abs(jv) + np.abs(jt) @ np.abs(v)
        assert abs(lam @ jv - jt @ v) <= 1e-13 * scale, i
