"""The headers that the FP64 kernels run and that host builds share (the regrouped right-hand sides,
their RK4 step and its transpose, checkpoint slots, turns, interpolation weights) under
AddressSanitizer and UndefinedBehaviorSanitizer, driven by a small program of its own."""
import os

import pytest

from conftest import ROOT
from test_sanitizers import _build_and_run, _have

DRIVER = r"""
#include <cmath>
#include <cstdio>
#include <vector>
#include "checkpoint.hpp"
#include "grid_weights.hpp"
#include "ham_accel.hpp"
#include "kerr_accel.hpp"
#include "turns.hpp"
struct Half {
    double M, a, Ys[4][6];
    void operator()(int, double r, double th, double ut, double ur, double uth, double uph, double &at2,
                    double &ar, double &ath, double &aph2) const {
        const double s = std::sin(th), c = std::cos(th);
        if (a == 0.0)
            malbec::schwarzschild_accel_half<double>(M, r, s * s, s * c, ut, ur, uth, uph, at2, ar, ath, aph2);
        else malbec::kerr_accel_half<double>(M, a, r, s * s, s * c, ut, ur, uth, uph, at2, ar, ath, aph2);
    }
    double &Y(int st, int k) { return Ys[st][k]; }
    void keep() const {}
    void prepare(int, double) const {}
    void vjp(int, double r, double th, double ut, double ur, double uth, double uph, double bt, double br,
             double bh, double bp, double &rb, double &thb, double ub[4]) const {
        const double s = std::sin(th), c = std::cos(th);
        malbec::kerr_accel_half_vjp<double>(M, a, r, s * s, s * c, ut, ur, uth, uph, bt, br, bh, bp, rb, thb, ub);
    }
};
struct Ham {
    double M, a;
    malbec::HamConst<double> P;
    void operator()(int, double r, double th, double pr, double pth, double &dt, double &dr, double &dth,
                    double &dph, double &dpr, double &dpth) const {
        const double s = std::sin(th), c = std::cos(th);
        if (a == 0.0)
            malbec::schwarzschild_ham_s2<double>(M, r, s * s, s * c, pr, pth, P, dt, dr, dth, dph, dpr, dpth);
        else malbec::kerr_ham_s2<double>(M, a, r, s * s, s * c, pr, pth, P, dt, dr, dth, dph, dpr, dpth);
    }
};
int main() {
    double s = 0.0;
    for (double a : {0.9, 0.0}) {
        double y[8] = {0.0, 9.0, 1.2, 0.0, 1.1, 0.05, 0.01, 0.03}, y1[8], sr[3];
        double z[8] = {0.0, 9.0, 1.2, 0.0, -0.95, 0.05, 0.3, 3.0}, z1[8];
        std::vector<double> slots(8 * (200 / 64 + 1));
        int64_t k0 = 0;
        for (int part = 0; part < 2; ++part, k0 += 100)
            malbec::run_checkpointed((int32_t)k0, 100, 64, 200 / 64, true,
                [&](int32_t m, bool &active) {
                    for (int32_t i = 0; i < m; ++i) {
                        Half f{1.0, a, {}};
                        malbec::rk4_step_half(f, 0.02, y, y1, sr);
                        double lam[8] = {1, 2, 3, 4, 5, 6, 7, 8};
                        malbec::rk4_vjp_half(f, 0.02, y, lam);
                        Ham h{1.0, a, malbec::ham_const(a, z[4], z[7])};
                        malbec::rk4_ham_step(h, 0.02, z, z1, sr);
                        for (int k = 0; k < 8; ++k) { s += lam[k] + z1[k]; y[k] = y1[k]; z[k] = z1[k]; }
                    }
                    active = true;
                    return m;
                },
                [&](int32_t slot) { for (int k = 0; k < 8; ++k) slots.at(8 * slot + k) = y[k]; });
        for (double x : slots) s += x;
    }
    for (int32_t m : {0, 1, 255, 256, 257, 569, 4095}) {
        std::vector<int> had_work(m > 0 ? m : 1);
        const int32_t turns = malbec::turns_of_block(1000, 16, m);
        for (int t = 0; t < 256; ++t) {
            int32_t j = t, had = 0;
            for (int32_t turn = 0; turn < turns; ++turn) {
                if (j < m) had_work.at(j) += malbec::steps_of_turn(1000, 16, had);
                malbec::next_turn(m, j, had);
            }
        }
        s += had_work[0] + malbec::turns_of_block(2147483647, 16, m) % 7 + malbec::turns_per_cu(m * 1000LL, 256, 1000);
    }
    double w[4], d[4];
    for (int k = 0; k < 100; ++k) { malbec::lagrange4(0.01 * k, w, d); s += w[0] + d[3]; }
    std::printf("ok %.6f\n", s);
    return std::isfinite(s) ? 0 : 3;
}
"""


@pytest.mark.skipif(not _have("g++"), reason="g++ not found")
def test_fp64_kernel_headers_under_address_and_undefined_sanitizers(tmp_path):
    _build_and_run(tmp_path, "g++", "fp64_headers_driver.cpp", DRIVER,
                   ["-std=c++17", "-I", os.path.join(ROOT, "paper_1803_08320_amd", "csrc")])
