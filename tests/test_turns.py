"""Launches in turns (csrc/turns.hpp): the turns of a block compiled for the host with undefined
behaviour trapped, and the kernels with the largest number of steps, ended by their lanes."""
import ctypes as C
import math
import os
import subprocess

import pytest

from conftest import ROOT

MAX = 2**31 - 1

SRC = r"""
#include <vector>
#include "turns.hpp"
extern "C" int32_t per_cu(int64_t n, int64_t steps) { return malbec::turns_per_cu(n, 256, steps); }
extern "C" int32_t turn_count(int32_t n_steps, int32_t q, int32_t m) { return malbec::turns_of_block(n_steps, q, m); }
extern "C" int32_t steps_after(int32_t n_steps, int32_t q, int32_t had) { return malbec::steps_of_turn(n_steps, q, had); }
// The turns of a block, lane k stopping after stop(k) = k * stride steps (stride < 0: never).  0 when
// every lane has had its steps, none of them twice in a turn, and the block has left in time.
extern "C" int play(int32_t n_steps, int32_t q, int32_t m, int32_t stride) {
    std::vector<int64_t> got(m, 0), turn_of(m, -1);
    int32_t j[256], had[256], worked = 0, turn = 0;
    for (int t = 0; t < 256; ++t) { j[t] = t; had[t] = 0; }
    auto end = [&](int k) { return stride < 0 || (int64_t)k * stride > n_steps ? (int64_t)n_steps : (int64_t)k * stride; };
    const int32_t turns = malbec::turns_of_block(n_steps, q, m);
    for (; turn < turns; ++turn) {
        for (int t = 0; t < 256; ++t) {
            const int32_t steps = malbec::steps_of_turn(n_steps, q, had[t]);
            if (j[t] < m && steps > 0 && got[j[t]] < end(j[t])) {
                if (turn_of[j[t]] == turn) return 1;
                worked = turn_of[j[t]] = turn;
                got[j[t]] = got[j[t]] + steps < end(j[t]) ? got[j[t]] + steps : end(j[t]);
            }
            malbec::next_turn(m, j[t], had[t]);
        }
        if (malbec::look_after(turn) && worked <= turn - malbec::kIdleTurns) break;
    }
    for (int k = 0; k < m; ++k)
        if (got[k] != end(k)) return 2;
    return turn <= worked + 2 * malbec::kIdleTurns ? 0 : 3;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("turns")
    src, so = d / "turns.cpp", d / "libturns.so"
    src.write_text(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fsanitize=undefined",
                    "-fsanitize-undefined-trap-on-error", "-I",
                    os.path.join(ROOT, "paper_1803_08320_amd", "csrc"), str(src), "-o", str(so)], check=True)
    lib = C.CDLL(str(so))
    lib.per_cu.argtypes = [C.c_int64, C.c_int64]
    return lib


@pytest.mark.parametrize("m", [0, 1, 255, 256, 257, 300, 396, 511, 512, 513, 569, 2275, 4095])
@pytest.mark.parametrize("q", [16, 32])
def test_every_lane_has_its_steps(host, q, m):
    for n_steps in (100, 101, 127, 128, 1000):
        assert host.play(n_steps, q, m, -1) == 0, n_steps
    # a step count far beyond what the lanes take
    for stride in (0, 1, 3):
        assert host.play(MAX, q, m, stride) == 0, stride


@pytest.mark.parametrize("m", [1, 256, 257, 569, 2275])
@pytest.mark.parametrize("q", [16, 32])
def test_turns_of_the_longest_calls(host, q, m):
    for n_steps in (MAX, MAX - 1, MAX - q + 2, MAX - 40):
        runs = -(-n_steps // q)
        assert host.turn_count(n_steps, q, m) == (-(-runs * m // 256) if m >= 256 else runs)
        # the last turns of a lane, and the turn after them
        assert host.steps_after(n_steps, q, runs - 2) == q
        assert 0 < host.steps_after(n_steps, q, runs - 1) == n_steps - (runs - 1) * q
        assert host.steps_after(n_steps, q, runs) == host.steps_after(n_steps, q, runs + 1) == 0


@pytest.mark.parametrize("w,most,blocks", [(1, 0.55, 1), (2, 0.6, 2), (3, 0.6, 3), (4, 0.6, 4), (5, 0.6, 4),
                                           (6, 0.45, 4), (7, 0.3, 4), (8, 0.3, 4)])
def test_rule_at_its_limits(host, w, most, blocks):
    """A whole number of levels and the lanes beyond the limit take one thread per lane, between them the
    launch is in turns, from 100 steps on; the blocks that are resident fit the LDS."""
    level = 256 * 256
    last = w * level + int(most * level)
    assert host.per_cu(w * level, 1000) == 0
    assert host.per_cu(w * level + 1, 100) == blocks
    assert host.per_cu(last, 2**31 - 1) == blocks
    assert host.per_cu(last + 1, 1000) == 0
    assert host.per_cu(w * level + 1, 99) == 0
    share = -(-last // (256 * blocks))
    assert share <= 16 * 256 and min(blocks, 3) * (share * 76 + 2064) <= 160 * 1024


def test_rule_outside_its_range(host):
    for n in (0, 1, 65535, 9 * 65536 + 1, 20 * 65536 + 5, 2**40):
        assert host.per_cu(n, 1000) == 0


def inward_and_outward(m, n, formulation):
    """A Kerr batch none of whose lanes is active after 400 steps."""
    st = [(1.0, 0.9)]
    state, _, _ = m.init_particles(m.ICSpec(mode=m.IC_CONSTANTS, seed=6), st, n)
    state[5] = -30.0
    state[5, ::3] = 30.0
    state[6, 5::1013] = float("nan")
    if formulation == "hamiltonian":
        m.convert_state(state, st, True)
    status, steps = m.new_lane_arrays(n)
    status[11::501] = 2
    return st, state, status, steps


@pytest.mark.gpu
@pytest.mark.parametrize("formulation", ["christoffel", "hamiltonian"])
@pytest.mark.parametrize("n", [65537, 131072 + 77, 300007])
def test_longest_call_ends_with_its_lanes(formulation, n):
    """2^31 - 1 steps, the cap of a run until every lane stops, in turns (block = 0) and with one
    thread per lane: the same bits, and no block goes on after its last lane."""
    import torch

    import paper_1803_08320_amd as m
    st, state, status0, steps0 = inward_and_outward(m, n, formulation)
    kw = dict(h=0.02, r_escape=60.0, formulation=formulation)
    s, a, b = state.clone(), status0.clone(), steps0.clone()
    m.integrate(s, a, b, st, n_steps=400, block=256, **kw)
    assert not bool((a == 0).any())  # so the calls below end
    for block in (256, 0):
        s2, a2, b2 = state.clone(), status0.clone(), steps0.clone()
        m.integrate(s2, a2, b2, st, n_steps=MAX, block=block, **kw)
        for x, y in ((s, s2), (a, a2), (b, b2)):
            assert torch.equal(x.view(torch.int64) if x.dtype == torch.float64 else x,
                               y.view(torch.int64) if y.dtype == torch.float64 else y), block


@pytest.mark.gpu
@pytest.mark.parametrize("node_dtype", ["float64", "float32"])
@pytest.mark.parametrize("n", [65537, 131072 + 77])
def test_longest_gridded_call_ends_with_its_lanes(node_dtype, n):
    import torch

    import paper_1803_08320_amd as m
    g = m.grid_kerr(1.0, 0.9, 401, 201, 1.5, 60.0 / 400, 0.1, (math.pi - 0.2) / 200, 1.72,
                    node_dtype=getattr(torch, node_dtype))
    _, state, status0, steps0 = inward_and_outward(m, n, "hamiltonian")
    s, a, b = state.clone(), status0.clone(), steps0.clone()
    m.integrate_grid(s, a, b, g, 0.02, 400, 55.0, block=256)
    assert not bool((a == 0).any())
    for block in (256, 0):
        s2, a2, b2 = state.clone(), status0.clone(), steps0.clone()
        m.integrate_grid(s2, a2, b2, g, 0.02, MAX, 55.0, block=block)
        for x, y in ((s, s2), (a, a2), (b, b2)):
            assert torch.equal(x.view(torch.int64) if x.dtype == torch.float64 else x,
                               y.view(torch.int64) if y.dtype == torch.float64 else y), block
