"""Index arithmetic of the checkpoint slots (csrc/checkpoint.hpp), compiled for the host with
undefined behaviour trapped, and the kernel that uses it."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from conftest import ROOT

MAX = 2**31 - 1

SRC = r"""
#include "checkpoint.hpp"
extern "C" int32_t segments(int32_t n_steps, int32_t every) { return malbec::checkpoint_segments(n_steps, every); }
// A lane that stops after `stop` steps of the call, from launch to launch of `chunk` steps.  put_at[s]
// receives the step whose state slot s holds.  Returns the steps taken, negative: a run of no steps or
// of more than the launch has left, or a slot outside the call's.
extern "C" int64_t walk(int64_t n_steps, int64_t chunk, int32_t every, int64_t stop, int64_t *put_at) {
    int64_t at = 0, bad = 0;
    const int32_t last = (int32_t)(n_steps / every);
    for (int64_t k0 = 0; k0 < n_steps; k0 += chunk) {
        const int32_t n = (int32_t)(n_steps - k0 < chunk ? n_steps - k0 : chunk);
        int64_t left = n;
        at += malbec::run_checkpointed(
            (int32_t)k0, n, every, last, at == k0 && at < stop,
            [&](int32_t m, bool &active) {
                if (m < 1 || m > left) { bad = -1; active = false; return 0; }
                const int64_t done = at + (n - left), take = m < stop - done ? m : stop - done;
                left -= take;
                active = done + take < stop;
                return (int32_t)take;
            },
            [&](int32_t s) {
                if (s < 0 || s > last) bad = -2;
                else put_at[s] = at + (n - left);
            });
        if (bad) return bad;
    }
    return at;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    src, so = d / "slots.cpp", d / "libslots.so"
    src.write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-fsanitize=undefined",
                    "-fsanitize-undefined-trap-on-error", "-I",
                    os.path.join(ROOT, "paper_1803_08320_amd", "csrc"), str(src), "-o", str(so)], check=True)
    lib = C.CDLL(str(so))
    lib.walk.restype = C.c_int64
    lib.walk.argtypes = [C.c_int64, C.c_int64, C.c_int32, C.c_int64, C.POINTER(C.c_int64)]
    return lib


@pytest.mark.parametrize("every", [1, 7, 50, 64, 100, 101, 2**30, 2**30 + 1, MAX - 50, MAX - 1, MAX])
@pytest.mark.parametrize("n_steps,chunk", [(1, 1), (100, 100), (100, 50), (100, 33), (101, 64)])
def test_every_slot_holds_its_step(host, every, n_steps, chunk):
    for stop in (0, 1, 49, 50, 51, 99, 100, 10**6):
        slots = n_steps // every + 1
        at = (C.c_int64 * slots)(*[-1] * slots)
        taken = host.walk(n_steps, chunk, every, stop, at)
        assert taken == min(stop, n_steps), (stop, taken)
        assert list(at) == [min(s * every, stop) for s in range(slots)], stop


@pytest.mark.parametrize("n_steps,chunk", [(MAX, MAX), (MAX, 2**30 + 7), (MAX - 1, MAX - 1)])
@pytest.mark.parametrize("every", [2**29 + 1, 2**30, MAX - 1, MAX])
def test_slots_of_the_longest_calls(host, every, n_steps, chunk):
    for stop in (5, 2**30, MAX - 2, 2**40):
        slots = n_steps // every + 1
        at = (C.c_int64 * slots)(*[-1] * slots)
        assert host.walk(n_steps, chunk, every, stop, at) == min(stop, n_steps)
        assert list(at) == [min(s * every, stop) for s in range(slots)]


@pytest.mark.parametrize("every", [1, 2, 50, 99, 100, 101, 2**30, MAX - 99, MAX])
def test_segments_of_the_walk_back(host, every):
    for n_steps in (1, 2, 100, MAX - 1, MAX):
        assert host.segments(n_steps, every) == -(-n_steps // every)


@pytest.mark.gpu
@pytest.mark.parametrize("every", [2**31 - 50, MAX])
def test_first_state_only(every):
    """checkpoint_every beyond the call, over several launches: slot 0 is the initial state and the
    result that of the same call without checkpoints."""
    import torch

    import paper_1803_08320_amd as m
    n, st = 300, [(1.0, 0.9)]
    y0, _, _ = m.init_particles(m.ICSpec(mode=m.IC_CONSTANTS, seed=2), st, n)
    out = []
    for k in (0, every):
        y, (status, steps) = y0.clone(), m.new_lane_arrays(n)
        ck = torch.full((1, 8, n), -1.0, dtype=torch.float64, device="cuda") if k else None
        m.integrate(y, status, steps, st, h=0.02, n_steps=100, steps_per_chunk=50, checkpoints=ck,
                    checkpoint_every=k)
        out.append((y, status, steps))
    assert torch.equal(ck[0], y0)
    for a, b in zip(*out):
        assert torch.equal(a, b)
    assert np.all(out[1][2].cpu().numpy() == 100)
