"""The CONSTANTS sampler on the boundary of the admissible draws."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def one(m, r, th, E, Lz, Q, a):
    """The state of the single draw (r, theta, E, L_z, Q), NaN when it is rejected."""
    spec = m.ICSpec(mode=m.IC_CONSTANTS, seed=1, r_range=(r, r), th_range=(th, th), E_range=(E, E),
                    Lz_range=(Lz, Lz), Q_range=(Q, Q), max_attempts=1)
    return m.init_particles(spec, [(1.0, a)], 1)[0][:, 0].cpu().numpy()


@pytest.mark.parametrize("where", ["between", "equator", "many turns"])
def test_decision_is_that_of_the_state(where):
    """Carter constants a few units in the last place around the polar turning point: the draws are
    accepted from some Q on, and every accepted state has Theta > 0 (u^theta != 0), except where Theta
    is exactly zero, at one Q at most."""
    import paper_1803_08320_amd as m
    rng = np.random.default_rng(1)
    crossed = 0
    for _ in range(40):
        th = rng.uniform(0.3, 2.8)
        if where == "equator":
            th = 0.5 * math.pi + rng.choice([-1, 1]) * 10.0 ** rng.uniform(-14, -4)
        elif where == "many turns":
            th += 2.0 * math.pi * rng.integers(100, 40000)
        E, Lz, a, r = rng.uniform(0.93, 1.2), rng.uniform(0.1, 3.0), rng.uniform(0, 1), rng.uniform(10, 14)
        turn = math.cos(th) ** 2 * (a * a * (1 - E * E) + Lz * Lz / math.sin(th) ** 2)
        q = [turn]
        for _ in range(5):
            q = [np.nextafter(q[0], -1.0)] + q + [np.nextafter(q[-1], 1e9)]
        states = [one(m, r, th, E, Lz, float(x), a) for x in q]
        accepted = [bool(np.isfinite(y).all()) for y in states]
        assert accepted == sorted(accepted), (th, accepted)
        assert sum(bool(y[6] == 0.0) for y, ok in zip(states, accepted) if ok) <= 1, (th, accepted)
        crossed += accepted[-1] and not accepted[0]
    assert crossed >= 5  # (others: R < 0, or a boundary more than five units from the host's)
