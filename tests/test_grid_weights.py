"""The interpolation weights of the gridded metric (csrc/grid_weights.hpp), compiled for the host,
against the same basis in extended precision."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from conftest import ROOT

SRC = r"""
#include <math.h>
#include "grid_weights.hpp"
extern "C" void weights(long n, const double *u, double *w, double *d6) {
    for (long i = 0; i < n; ++i) malbec::lagrange4(u[i], w + 4 * i, d6 + 4 * i);
}
"""
LD = np.longdouble


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("weights")
    src, so = d / "w.cpp", d / "libw.so"
    src.write_text(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", "-I",
                    os.path.join(ROOT, "paper_1803_08320_amd", "csrc"), str(src), "-o", str(so)], check=True)
    return C.CDLL(str(so))


def products(u, one):
    """Every weight from its own product, in the type of u."""
    um, u2, up, uu3 = u - one, u - 2 * one, u + one, 3 * u * u
    six, half = one / 6, one / 2
    w = [-u * um * u2 * six, up * um * u2 * half, -up * u * u2 * half, up * u * um * six]
    d = [-(uu3 - 6 * u + 2) * six, (uu3 - 4 * u - 1) * half, -(uu3 - 2 * u - 2) * half, (uu3 - 1) * six]
    return np.array(w), np.array(d)


@pytest.mark.parametrize("f", [lambda x: x * x, lambda x: 1 / x, lambda x: x * x / (x * x - 2 * x + 0.81),
                               lambda x: np.sqrt(1 - 2 / x)], ids=["r2", "1/r", "grr", "alpha"])
@pytest.mark.parametrize("x0,dx", [(1.5, 0.075), (1.5, 0.15), (4.0, 1.0)])
def test_values_and_derivatives_have_no_bias(host, f, x0, dx):
    """Over offsets as the kernel forms them, the error that the weights put into the value and the
    derivative of the metric's functions averages out (within five standard errors of the mean) and
    its rms is no larger than with every weight from its own product."""
    n = 200_000
    x = np.random.default_rng(3).uniform(6.0, 50.0, n)
    q = (x - x0) * (1.0 / dx)
    i = np.trunc(q)
    u = q - i
    w, d6 = np.zeros((n, 4)), np.zeros((n, 4))
    dp = C.POINTER(C.c_double)
    host.weights(C.c_long(n), u.ctypes.data_as(dp), w.ctypes.data_as(dp), d6.ctypes.data_as(dp))
    F = np.array([f(x0 + dx * (i - 1 + k)) for k in range(4)]).astype(LD)
    exact = products(u.astype(LD), LD(1))
    plain = products(u, 1.0)
    for got, ref, own in ((w.T.astype(LD), exact[0], plain[0]), (d6.T.astype(LD) / 6, exact[1], plain[1])):
        want = (ref * F).sum(0)
        err = ((got * F).sum(0) - want) / np.abs(want)
        rms = float(np.sqrt((err ** 2).mean()))
        own_rms = float(np.sqrt(((((own.astype(LD) * F).sum(0) - want) / want) ** 2).mean()))
        assert abs(float(err.mean())) <= 5 * rms / np.sqrt(n)
        assert rms <= own_rms


@pytest.mark.gpu
@pytest.mark.parametrize("f32", [False, True])
def test_stage_points_anywhere(orc, f32):
    """Momenta that carry the stage points off the grid by any distance, to infinity and to NaN: every
    gather stays inside the grid, and the lanes end as the oracle's, after the same number of steps (as
    HORIZON or as NONFINITE where the square of the momentum overflows, which the oracle forms in
    another order)."""
    import torch

    import paper_1803_08320_amd as m
    G = orc.grid_kerr(1.0, 0.6, 33, 17, 4.0, 0.5, 0.5, 0.13)
    nodes = G.nodes.astype(np.float32) if f32 else G.nodes
    G = orc.Grid(nodes.astype(np.float64), G.r0, G.dr, G.th0, G.dth)
    g = m.Grid(torch.as_tensor(nodes).cuda(), G.r0, G.dr, G.th0, G.dth, 4.6)
    vals = [s * v for v in (1.0, 1e2, 1e9, 3e9, 1e10, 1e20, 1e100, 1e154, 1e300) for s in (1, -1)]
    vals += [np.inf, -np.inf, np.nan]
    z = []
    for c in (4, 5, 6, 7):
        for v in vals:
            for r, th in ((4.7, 0.7), (9.0, 1.5), (18.0, 2.4)):
                y = np.array([0.0, r, th, 0.0, -0.95, 0.05, 0.3, 2.0])
                y[c] = v
                z.append(y)
    z = np.array(z).T.copy()
    state = torch.as_tensor(z).cuda()
    status, steps = m.new_lane_arrays(z.shape[1])
    m.integrate_grid(state, status, steps, g, 0.05, 20, 18.5)
    ref = orc.integrate_grid(G, z, 0.05, 20, r_stop=4.6, r_escape=18.5)
    got, huge = status.cpu().numpy(), ~(np.abs(z[4:]).max(axis=0) < 1e154)
    assert np.array_equal(got[~huge], ref[1][~huge])
    assert np.array_equal(got[huge] == 0, ref[1][huge] == 0)
    assert np.array_equal(steps.cpu().numpy(), ref[2])
    assert set(np.unique(ref[1])) >= {0, 1, 4}
