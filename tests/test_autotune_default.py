"""The autotuner never makes a launch slower than the library's default shape."""
import json

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture
def tuner(tmp_path, monkeypatch):
    import paper_1803_08320_amd as m
    from paper_1803_08320_amd import autotune
    monkeypatch.setenv("MALBEC_TUNE_CACHE", str(tmp_path / "tune.json"))
    launched = []
    make = m.c_run

    def c_run(*a):
        run = make(*a)
        launched.append((run.block, run.steps_per_chunk))
        return run
    monkeypatch.setattr(m, "c_run", c_run)
    return m, autotune, launched, tmp_path / "tune.json"


def lanes(m, n):
    st = [(1.0, 0.9)]
    return st, m.init_particles(m.ICSpec(mode=m.IC_CONSTANTS, seed=2), st, n)[0]


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("gain,taken", [(0.9, True), (0.99, False)])
def test_explicit_shape_only_where_it_is_faster(tuner, monkeypatch, persistent, gain, taken):
    """The default is among the candidates, timed as the default also when an entry is there already, and an
    explicit shape has to beat it by more than the noise."""
    m, autotune, launched, path = tuner
    n = 3000
    st, s0 = lanes(m, n)
    shape = (128, 32 if persistent else 0)
    real = autotune._time

    def timed(fn, reps=2):
        del launched[:]
        real(fn, 1)
        assert len(set(launched)) == 1
        return gain if launched[0] == shape else 1.0
    monkeypatch.setattr(autotune, "_time", timed)
    for refresh in (False, True):
        got = autotune.integrate_shape(s0, st, 0.02, persistent=persistent, probe_steps=5, refresh=refresh)
        assert got == (shape if taken else (0, 0))
        del launched[:]
        status, steps = m.new_lane_arrays(n)
        m.integrate(s0.clone(), status, steps, st, h=0.02, n_steps=5, persistent=persistent)
        assert launched == [shape if taken else (0, 0)]


def test_lane_counts_that_may_run_in_turns_keep_the_default(tuner):
    """A cached explicit shape of a size bucket is taken for its even lane counts alone, and an entry tuned
    without the default among the candidates not at all."""
    import torch
    m, autotune, launched, path = tuner
    level = 256 * torch.cuda.get_device_properties(0).multi_processor_count

    def launch(n, **kw):
        st, s0 = lanes(m, n)
        status, steps = m.new_lane_arrays(n)
        del launched[:]
        m.integrate(s0, status, steps, st, h=0.02, **{"n_steps": 100, **kw})
        return launched[0]

    for n, persistent, want in ((level + 500, False, (0, 0)), (level + 500, True, (0, 0)),
                                (2 * level, False, (64, 0)), (2 * level, True, (64, 8)),
                                (level + (9 * level) // 10, False, (64, 0)), (4 * level + 1, False, (0, 0)),
                                (4 * level + 1, True, (64, 8))):
        e = {"block": 64, "chunk": 8 if persistent else 0, "ms": {"0,0": 2.0, "64,8": 1.0}}
        key = autotune._integrate_key(n, 1, "f64", "christoffel", persistent)
        autotune._store({key: e})
        assert launch(n, persistent=persistent) == want, n
        assert json.loads(path.read_text())[key]["block"] == 64
        del e["ms"]["0,0"]
        autotune._store({key: e})
        assert launch(n, persistent=persistent) == (0, 0), n
    autotune._store({autotune._integrate_key(level + 500, 1, "f64", "christoffel", False):
                     {"block": 64, "chunk": 0, "ms": {"0,0": 2.0, "64,0": 1.0}}})
    assert launch(level + 500, n_steps=99) == (64, 0)          # too few steps for turns
    assert launch(level + 500, n_steps=1000, steps_per_chunk=50) == (64, 50)
    assert launch(level + 500, n_steps=200, steps_per_chunk=100) == (0, 100)
