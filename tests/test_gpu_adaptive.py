"""GPU parity of the adaptive Dormand-Prince 5(4) integrator against the oracle's
(same pair, same controller, same stop rules)."""
import math

import numpy as np
import pytest

from parity import TOL_F64, compare, mixed_rel

pytestmark = pytest.mark.gpu

KERR_RANGES = ((5.0, 50.0), (math.pi / 4, 3 * math.pi / 4), (0.92, 0.98), (2.5, 4.5), (0.0, 12.0))
CTL = dict(rtol=1e-9, atol=1e-9, fac=0.9, facmin=0.2, facmax=5.0)


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1803_08320_amd as m
    m.lib()
    return m


def to_dev(x, dtype=None):
    import torch
    return torch.as_tensor(np.ascontiguousarray(x), dtype=dtype).cuda()


def run_gpu(m, sts, s0, tau_end, h0, st_of_lane=None, **kw):
    import torch
    n = s0.shape[1]
    state = to_dev(s0, torch.float64)
    tau = torch.zeros(n, dtype=torch.float64, device="cuda")
    h = torch.full((n,), h0, dtype=torch.float64, device="cuda")
    status = torch.zeros(n, dtype=torch.int32, device="cuda")
    steps = torch.zeros(n, dtype=torch.int32, device="cuda")
    rej = torch.zeros(n, dtype=torch.int32, device="cuda")
    sol = None if st_of_lane is None else to_dev(st_of_lane, torch.int32)
    args = dict(CTL)
    args.update(kw)
    m.integrate_adaptive(state, tau, h, status, steps, rej, sts, tau_end, st_of_lane=sol, **args)
    torch.cuda.synchronize()
    return tuple(x.cpu().numpy() for x in (state, tau, h, status, steps, rej))


def key(steps, rej):
    """Accepted and rejected attempt counts as one integer (both must match)."""
    return steps.astype(np.int64) * 65536 + rej


def oracle(orc, sts, s0, tau_end, h0, **kw):
    args = dict(CTL)
    args.update(kw)
    return orc.integrate_adaptive(sts, s0, tau_end, h0, **args)


def check(orc, sts, s0, got, ref, tau_end, h0, **kw):
    """State, status and attempt counts per lane against the oracle, with the
    conditioning guard of parity.compare (an accept/reject decision taken at
    err ~ 1 can go either way under a change of rounding).  A lane that both sides
    stop as HORIZON ends next to the coordinate singularity at r_+ (u^t ~ 1/Delta;
    a 1-ulp change of r0 moves its final state by ~1e-8 in the oracle itself), so
    for those the status and the attempt counts are the comparison."""
    def rerun(p0):
        y, tau, h, st, sp, rj = oracle(orc, sts, p0, tau_end, h0, **kw)
        return y, st, key(sp, rj)
    both_hz = (got[3] == 1) & (ref[3] == 1)
    g0 = np.where(both_hz[None, :], ref[0], got[0])
    # end-of-interval splits: both sides active on tau_end with the same state (1e-10),
    # the same rejections and one accepted attempt more on one side.  The last attempt is
    # clipped to land on tau_end, and the two sides' step sizes differ by ~1e-5 relative
    # (err^(-1/5) of a cancelling difference), so the penultimate step can stop just
    # short of tau_end on one side (which then takes a sliver of a step) and reach it on
    # the other; such lanes are counted as ties.
    split = ((got[3] == 0) & (ref[3] == 0) & (got[1] == tau_end) & (ref[1] == tau_end)
             & (got[5] == ref[5]) & (np.abs(got[4].astype(np.int64) - ref[4]) == 1)
             & (mixed_rel(got[0], ref[0]) <= TOL_F64))
    gkey = np.where(split, key(ref[4], ref[5]), key(got[4], got[5]))
    stats = compare(orc, sts, s0, g0, got[3], gkey, ref[0], ref[3], key(ref[4], ref[5]), rerun)
    from conftest import PARITY_LOG
    PARITY_LOG.append("    (of them %d end-of-interval splits: one accepted attempt more on one side)"
                      % int(split.sum()))
    assert split.sum() <= max(2, 0.001 * split.size)
    same = (got[3] == ref[3]) & (got[4] == ref[4]) & (got[5] == ref[5])
    # the affine parameter lands exactly on tau_end for lanes still active
    act = same & (ref[3] == 0)
    assert np.array_equal(got[1][act], ref[1][act]) and np.all(ref[1][act] == tau_end)
    # h on return is the step suggested after the last accepted step, and that step is
    # clipped to tau_end - tau_prev.  Every step size follows err^(-1/5) of an
    # embedded difference whose rounding floor is ~1e-4 of its tolerance at rtol =
    # 1e-12, so the two sides' steps differ by up to a few 1e-5 relative and their sums
    # tau_prev by up to ~1.5e-5 tau_prev (both measured without clipping in
    # test_adaptive_full_size_sampled); the clipped step carries that difference
    # absolute, and the suggestion is at most facmax times the clipped step.  The
    # state, tau and the attempt counts above already fix every accept/reject decision
    # exactly.
    facmax = kw.get("facmax", CTL["facmax"])
    dh = np.abs(got[2][same] - ref[2][same])
    print("final h: max |dh| %.3e, max |dh|/h %.3e, median |dh|/h %.3e"
          % (dh.max(), (dh / np.abs(ref[2][same])).max(), np.median(dh / np.abs(ref[2][same]))))
    assert np.all(dh <= 1e-3 * np.abs(ref[2][same]) + facmax * 3e-5 * tau_end)
    assert np.median(dh / np.abs(ref[2][same])) <= 1e-4
    return stats


@pytest.mark.parametrize("persistent", [False, True])
def test_adaptive_parity_kerr(m, orc, persistent):
    st = [(1.0, 0.9)]
    rc, s0, _, _ = orc.ic_constants(71, st, 600, KERR_RANGES)
    got = run_gpu(m, st, s0, 300.0, 0.1, persistent=persistent)
    ref = oracle(orc, st, s0, 300.0, 0.1)
    assert ref[5].sum() > 0  # the controller rejects some attempts
    check(orc, st, s0, got, ref, 300.0, 0.1)


def test_adaptive_plunging_and_mixed_spins(m, orc):
    sts = [(1.0, 0.0), (1.0, 0.5), (1.0, 0.998)]
    n = 900
    st_of_lane = (np.arange(n) % 3).astype(np.int32)
    rc, s0, _, _ = orc.ic_constants(72, sts, n, KERR_RANGES, st_of_lane=st_of_lane)
    got = run_gpu(m, sts, s0, 2000.0, 0.05, st_of_lane=st_of_lane)
    for k in range(3):
        sel = np.flatnonzero(st_of_lane == k)
        ref = oracle(orc, [sts[k]], s0[:, sel], 2000.0, 0.05)
        sub = tuple(x[..., sel] for x in got)
        check(orc, [sts[k]], s0[:, sel], sub, ref, 2000.0, 0.05)
        if k == 0:
            assert (ref[3] == 1).sum() > 30  # Schwarzschild draws plunge


def test_persistent_equals_plain_bitwise_and_budget(m, orc):
    st = [(1.0, 0.7)]
    rc, s0, _, _ = orc.ic_constants(73, st, 1000, KERR_RANGES)
    a = run_gpu(m, st, s0, 500.0, 0.1, persistent=False)
    b = run_gpu(m, st, s0, 500.0, 0.1, persistent=True, steps_per_chunk=3)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    c = run_gpu(m, st, s0, 1e6, 0.1, max_attempts=7)
    assert np.all(c[3] == 5) and np.all(c[4] + c[5] == 7)
    ref = oracle(orc, st, s0, 1e6, 0.1, max_attempts=7)
    assert np.array_equal(ref[3], c[3])


def test_adaptive_full_size_sampled(m, orc):
    """The benchmark's adaptive launch: Kerr a = 0.9, 1,048,576 lanes to tau = 400 at
    rtol = atol = 1e-12 under the persistent queue in periapsis order.  8,192 strided lanes hold the
    oracle's own initial data (the device builder's agree with it to the rounding of
    sqrt(R)) and are compared with the oracle; over all lanes, active ones end on
    tau_end."""
    import torch
    st = [(1.0, 0.9)]
    n = 1 << 20
    spec = m.ICSpec(mode=m.IC_CONSTANTS, seed=2, r_range=KERR_RANGES[0], th_range=KERR_RANGES[1],
                    E_range=KERR_RANGES[2], Lz_range=KERR_RANGES[3], Q_range=KERR_RANGES[4])
    state, consts, _ = m.init_particles(spec, st, n)
    idx = np.arange(0, n, n // 8192)
    s0 = np.concatenate([orc.ic_constants(2, st, 1, KERR_RANGES, lane0=int(i))[1] for i in idx], axis=1)
    assert mixed_rel(state.cpu().numpy()[:, idx], s0).max() < 5e-13
    state[:, torch.as_tensor(idx, device="cuda")] = to_dev(s0, torch.float64)
    tau = torch.zeros(n, dtype=torch.float64, device="cuda")
    h = torch.full((n,), 0.1, dtype=torch.float64, device="cuda")
    status = torch.zeros(n, dtype=torch.int32, device="cuda")
    steps = torch.zeros(n, dtype=torch.int32, device="cuda")
    rej = torch.zeros(n, dtype=torch.int32, device="cuda")
    m.integrate_adaptive(state, tau, h, status, steps, rej, st, 400.0, rtol=1e-12, atol=1e-12,
                         persistent=True, schedule="periapsis")
    torch.cuda.synchronize()
    all_out = tuple(x.cpu().numpy() for x in (state, tau, h, status, steps, rej))
    got = tuple(x[..., idx] for x in all_out)
    kw = dict(rtol=1e-12, atol=1e-12)
    ref = oracle(orc, st, s0, 400.0, 0.1, **kw)
    check(orc, st, s0, got, ref, 400.0, 0.1, **kw)
    act = all_out[3] == 0
    assert act.mean() > 0.99 and np.all(all_out[1][act] == 400.0)
    # the same lanes without the clipped last step: a fixed budget of attempts towards a
    # distant tau_end (every lane ends as BUDGET); the step sizes and their sum tau
    # agree to the rounding floor of the error estimate
    x = to_dev(s0, torch.float64)
    k = s0.shape[1]
    tau = torch.zeros(k, dtype=torch.float64, device="cuda")
    h = torch.full((k,), 0.1, dtype=torch.float64, device="cuda")
    z = [torch.zeros(k, dtype=torch.int32, device="cuda") for _ in range(3)]
    m.integrate_adaptive(x, tau, h, z[0], z[1], z[2], st, 1e6, max_attempts=400, **kw)
    torch.cuda.synchronize()
    g = [t.cpu().numpy() for t in (tau, h, z[0], z[1], z[2])]
    ref = oracle(orc, st, s0, 1e6, 0.1, max_attempts=400, **kw)
    assert np.array_equal(g[2], ref[3])
    assert np.array_equal(g[3], ref[4]) and np.array_equal(g[4], ref[5])
    bud = ref[3] == 5
    assert bud.mean() > 0.95
    assert np.all(np.abs(g[0] - ref[1])[bud] <= 3e-5 * ref[1][bud])
    assert np.all(np.abs(g[1] - ref[2])[bud] <= 1e-3 * ref[2][bud])
    assert np.median(np.abs(g[0] - ref[1])[bud] / ref[1][bud]) <= 1e-6


def run_lanes(m, sts, s0, status, tau0, tau_end, st_of_lane=None, **kw):
    import torch
    n = s0.shape[1]
    out = [to_dev(s0, torch.float64), to_dev(tau0, torch.float64),
           torch.full((n,), 0.1, dtype=torch.float64, device="cuda"), to_dev(status, torch.int32),
           torch.zeros(n, dtype=torch.int32, device="cuda"),
           torch.zeros(n, dtype=torch.int32, device="cuda")]
    sol = None if st_of_lane is None else to_dev(st_of_lane, torch.int32)
    args = dict(CTL)
    args.update(kw)
    m.integrate_adaptive(*out, sts, tau_end, st_of_lane=sol, **args)
    torch.cuda.synchronize()
    return tuple(x.cpu().numpy() for x in out)


def skipped_lanes(n, sol=None):
    """Lanes the integrator does not load: not ACTIVE, tau already at tau_end, or a bad
    spacetime index."""
    status = np.zeros(n, np.int32)
    status[3::97] = 1
    status[7::101] = 4
    tau0 = np.zeros(n)
    tau0[5::89] = 500.0
    if sol is not None:
        sol = sol.copy()
        sol[11::103] = 7
    return status, tau0, sol


def test_periapsis_schedule_gives_the_same_results(m, orc):
    """The periapsis order changes when lanes are handed out, not what they compute: the
    results are bitwise those of the index order and of the plain kernel, on three spins
    in one launch with inactive lanes, lanes already at tau_end, lanes with a bad
    spacetime index, plunging lanes, and a ragged tail."""
    sts = [(1.0, 0.0), (1.0, 0.5), (1.0, 0.9)]
    n = 3001
    sol = (np.arange(n) % 3).astype(np.int32)
    rc, s0, _, _ = orc.ic_constants(91, sts, n, KERR_RANGES, st_of_lane=sol)
    status, tau0, sol = skipped_lanes(n, sol)
    a = run_lanes(m, sts, s0, status, tau0, 300.0, sol, persistent=True, schedule="index")
    b = run_lanes(m, sts, s0, status, tau0, 300.0, sol, persistent=True, schedule="periapsis",
                  steps_per_chunk=5)
    c = run_lanes(m, sts, s0, status, tau0, 300.0, sol, persistent=False)
    for x, y, z in zip(a, b, c):
        assert np.array_equal(x, y) and np.array_equal(x, z)
    st = a[3]
    assert (st == 1).sum() > 30 and np.all(st[11::103][status[11::103] == 0] == 4)
    assert np.array_equal(a[0][:, 5::89], s0[:, 5::89])


def periapsis_key(M, a, E, L, Q, mu2, r0, status, tau0, tau_end):
    """The key of malbec_adaptive_order written out: the bucket j of the first zero of
    Carter's radial function R inward from r0 on r_j = r_+ 2^(j/32)."""
    if status != 0 or not tau0 < tau_end:
        return 1023
    rp = M + math.sqrt(M * M - a * a)

    def neg(j):
        r = rp * 2.0 ** (j / 32.0)
        D = r * r - 2 * M * r + a * a
        P = E * (r * r + a * a) - a * L
        return P * P - D * (mu2 * r * r + (L - a * E) ** 2 + Q) < 0.0
    x = 32.0 * math.log2(r0 / rp)
    if not x >= 1.0:
        return 1023
    j = int(min(x, 1022.0))
    while j > 0 and not neg(j):
        j -= 1
    return j


def test_periapsis_order_is_a_sorted_permutation(m, orc):
    """malbec_adaptive_order on 5,003 Kerr lanes: a permutation of the lanes whose keys
    do not decrease; skipped lanes take the last key; the keys are the periapsis
    buckets computed here from the oracle's constants of the same states (a key decided
    by the sign of R at a grid point may differ where R is within rounding of zero)."""
    import torch
    M, a = 1.0, 0.9
    sts = [(M, a)]
    n = 5003
    rc, s0, _, _ = orc.ic_constants(92, sts, n, KERR_RANGES)
    status, tau0, _ = skipped_lanes(n)
    order, keys = m.adaptive_order(to_dev(s0, torch.float64), to_dev(tau0, torch.float64),
                                   to_dev(status, torch.int32), sts, 400.0)
    o = order.cpu().numpy().astype(np.int64) & 0xFFFFFFFF
    k = keys.cpu().numpy().astype(np.int64) & 0xFFFFFFFF
    assert np.array_equal(np.sort(o), np.arange(n))
    assert np.all(np.diff(k[o]) >= 0)
    inv = orc.invariants(sts, s0)
    want = np.array([periapsis_key(M, a, inv[0, i], inv[1, i], inv[2, i], -inv[3, i], s0[1, i],
                                   status[i], tau0[i], 400.0) for i in range(n)])
    skip = (status != 0) | (tau0 >= 400.0)
    assert np.all(k[skip] == 1023) and skip.sum() > 100
    agree = k == want
    assert agree.mean() >= 0.999, np.flatnonzero(~agree)[:10]
    # a bound lane's periapsis lies inside its radius
    bound = (k > 0) & (k < 1023) & ~skip
    assert bound.mean() > 0.5
    rp = M + math.sqrt(M * M - a * a)
    assert np.all(rp * 2.0 ** (k[bound] / 32.0) <= s0[1][bound])


def test_periapsis_key_of_circular_orbits(m, orc):
    """On an equatorial circular orbit R has a double zero at the orbit's radius (R =
    R' = 0 there, Sections 3-4), so the periapsis is r0 itself: the key is the bucket
    that holds r0 or the one below it."""
    import torch
    M, a = 1.0, 0.9
    s0 = orc.ic_circular(93, M, a, 257, 4.0, 40.0, 0.0)
    n = s0.shape[1]
    z = np.zeros(n)
    order, keys = m.adaptive_order(to_dev(s0, torch.float64), to_dev(z, torch.float64),
                                   to_dev(np.zeros(n, np.int32), torch.int32), [(M, a)], 10.0)
    k = keys.cpu().numpy().astype(np.int64)
    j0 = np.floor(32.0 * np.log2(s0[1] / (M + math.sqrt(M * M - a * a)))).astype(np.int64)
    assert np.all((k == j0) | (k == j0 - 1)), np.c_[k, j0][k - j0 < -1][:5]


def test_periapsis_key_brackets_the_closest_approach(m, orc):
    """The key is the periapsis bucket, checked against the orbit itself: 24 bound Kerr
    lanes are integrated by the oracle (RK4, h = 0.05, radius sampled every 0.5 in tau)
    over more than a radial period, and the smallest radius each reaches lies in the
    lane's bucket, r_+ 2^(k/32) < r_min <= r_+ 2^((k+1)/32) (the sampled minimum is at
    most ~0.1 % above the true one)."""
    import torch
    M, a = 1.0, 0.9
    sts = [(M, a)]
    ranges = ((6.0, 14.0),) + KERR_RANGES[1:]
    rc, s0, _, _ = orc.ic_constants(94, sts, 24, ranges)
    n = s0.shape[1]
    z = np.zeros(n)
    order, keys = m.adaptive_order(to_dev(s0, torch.float64), to_dev(z, torch.float64),
                                   to_dev(np.zeros(n, np.int32), torch.int32), sts, 10.0)
    k = keys.cpu().numpy().astype(np.int64)
    y, st = s0.copy(), np.zeros(n, np.int32)
    rmin = y[1].copy()
    for _ in range(4000):  # tau = 2,000
        y, st, _ = orc.integrate(sts, y, 0.05, 10, status=st)
        rmin = np.minimum(rmin, np.where(st == 0, y[1], np.inf))
    bound = (st == 0) & (k > 0) & (k < 1023)
    assert bound.sum() >= 16
    rp = M + math.sqrt(M * M - a * a)
    lo = rp * 2.0 ** (k / 32.0)
    hi = rp * 2.0 ** ((k + 1) / 32.0)
    assert np.all(lo[bound] < rmin[bound]), np.c_[lo, rmin, hi][bound][:5]
    assert np.all(rmin[bound] <= hi[bound] * 1.002), np.c_[lo, rmin, hi][bound][:5]


@pytest.mark.parametrize("n,tau_end", [(1, 300.0), (257, 1e-3), (700, 2000.0)])
def test_length_order_of_unusual_lanes(m, orc, n, tau_end):
    """The estimate behind the work order meets plunging, escaping, null, unbound and unusable
    lanes, other masses, a tau_end below the first step and one beyond the steps it follows:
    every lane is handed out once and the results are bitwise those of the index order."""
    sts = [(1.0, 0.9), (2.5, 0.0), (1e-3, 1e-3)]
    sol = (np.arange(n) % 3).astype(np.int32)
    rc, s0, _, _ = orc.ic_constants(93, sts[:1], n, KERR_RANGES)
    M = np.array([x[0] for x in sts])[sol]
    s0[1] *= M
    s0[6:] /= M
    s0[5, 3::7] *= -40.0                   # inward or outward at high speed (norm not kept)
    s0[4:, 4::11] = [[1.4], [0.2], [0.0], [0.0]]
    s0[5, 6::50] = np.nan
    s0[1, 9::60] = 0.5 * M[9::60]          # inside the horizon
    status, tau0 = np.zeros(n, np.int32), np.zeros(n)
    kw = dict(r_escape=60.0, max_attempts=3000)
    a = run_lanes(m, sts, s0, status, tau0, tau_end, sol, persistent=True, schedule="index", **kw)
    b = run_lanes(m, sts, s0, status, tau0, tau_end, sol, persistent=True, schedule="periapsis", **kw)
    for x, y in zip(a, b):
        assert np.array_equal(x, y, equal_nan=x.dtype.kind == "f")
    if n > 500:
        assert len(np.unique(a[3])) >= 4   # several ways of ending are among them
