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
extern "C" int64_t turn_count(int32_t n_steps, int32_t q, int32_t m) { return malbec::turns_of_block(n_steps, q, m); }
extern "C" int32_t steps_after(int32_t n_steps, int32_t q, int32_t had) { return malbec::steps_of_turn(n_steps, q, had); }
// All turns of a block: 0 when every lane has had n_steps steps, none of them twice in a turn.
extern "C" int play(int32_t n_steps, int32_t q, int32_t m) {
    std::vector<int64_t> got(m, 0), turn_of(m, -1);
    int32_t j[256], had[256];
    for (int t = 0; t < 256; ++t) { j[t] = t; had[t] = 0; }
    const int64_t turns = malbec::turns_of_block(n_steps, q, m);
    for (int64_t turn = 0; turn < turns; ++turn)
        for (int t = 0; t < 256; ++t) {
            const int32_t steps = malbec::steps_of_turn(n_steps, q, had[t]);
            if (j[t] < m && steps > 0) {
                if (turn_of[j[t]] == turn) return 1;
                turn_of[j[t]] = turn;
                got[j[t]] += steps;
            }
            malbec::next_turn(m, j[t], had[t]);
        }
    for (int k = 0; k < m; ++k)
        if (got[k] != n_steps) return 2;
    return 0;
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
    lib.turn_count.restype = C.c_int64
    return lib


@pytest.mark.parametrize("m", [0, 1, 255, 256, 257, 300, 396, 511, 512, 513, 569, 2275])
@pytest.mark.parametrize("q", [16, 32])
def test_every_lane_has_its_steps(host, q, m):
    for n_steps in (100, 101, 127, 128, 1000):
        assert host.play(n_steps, q, m) == 0, n_steps


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
