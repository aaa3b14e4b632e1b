"""Performance cases: the work that a program has this library do, through its Python
entry points, from one handful of orbits to a full batch.

A case is a dict of plain values; `kind` says which entry points it goes through:

  orbits    integrate: fixed-step RK4 (FP64 or FP32-compensated, either formulation,
            plain or persistent launch, one spacetime or a batch of several spins)
  monitored integrate_monitored: the same with the invariant monitor in the step loop
  record    integrate_record: the same with the (tau, t, x, y, z) output stream
  adaptive  integrate_adaptive: Dormand-Prince 5(4), periapsis-ordered work queue
  grid      integrate_grid: a numerical 3+1 metric sampled on an (r, theta) grid
  camera    trace_camera: an image of a black hole with a thin disk
  gradient  IntegrateFromParams: a training step, forward and discrete adjoint
  setup     init_particles, convert_state and invariants: the start of every run

The library integrates in place; a pass therefore starts from a copy of the initial
state, as a program does that keeps its initial conditions.  `exact` is the same
discrete method in plain torch double precision (metric, right-hand sides, Runge-Kutta
tableaus and stop rules written out here).
"""
import math

import torch

import paper_1803_08320_amd as m

DEV = "cuda"
F64 = torch.float64
HORIZON_FACTOR = 1.01
R_ESCAPE = 1500.0
ACTIVE, HORIZON, ESCAPE, DISK, NONFINITE = 0, 1, 2, 3, 4
# the random bound orbits of the benchmark: ranges of r0, theta0, E, L_z and Carter's Q
R_RANGE, TH_RANGE = (5.0, 50.0), (0.25 * math.pi, 0.75 * math.pi)
E_RANGE, L_RANGE, Q_RANGE = (0.92, 0.98), (2.5, 4.5), (0.0, 12.0)


def listed():
    return [
        # one figure's worth of orbits for a few steps: launch latency and host path
        dict(name="few_orbits", kind="orbits", n=96, steps=16, h=0.1, a=0.9, spins=1, ic="bound",
             form="christoffel", precision="f64", persistent=False),
        # the Schwarzschild workload: 1,024 near-circular orbits, far too few to fill the chip
        dict(name="schwarzschild_1024", kind="orbits", n=1024, steps=2000, h=0.01, a=0.0, spins=1,
             ic="circular", form="christoffel", precision="f64", persistent=False),
        # the benchmark's batch of bound Kerr orbits (a tenth of its steps fill a pass)
        dict(name="kerr_1m", kind="orbits", n=1048576, steps=1000, h=0.02, a=0.9, spins=1, ic="bound",
             form="christoffel", precision="f64", persistent=False),
        # the paper's canonical form on a batch of no round size
        dict(name="hamiltonian_ragged", kind="orbits", n=300007, steps=1000, h=0.02, a=0.7, spins=1,
             ic="bound", form="hamiltonian", precision="f64", persistent=False),
        # a survey over 16 spins, FP32-compensated on the persistent queue
        dict(name="spins_f32k", kind="orbits", n=262144, steps=2000, h=0.02, a=0.99, spins=16,
             ic="bound", form="christoffel", precision="f32k", persistent=True),
        # trajectories for plotting: a record every 20 steps
        dict(name="record_ragged", kind="record", n=100003, steps=1000, every=20, h=0.02, a=0.9,
             form="christoffel"),
        # the adaptive integrator at the benchmark's tolerance
        dict(name="adaptive", kind="adaptive", n=262144, tau=400.0, tol=1e-12, a=0.9),
        # a numerical metric on the benchmark's 801 x 401 grid, and a coarser one in single precision
        dict(name="grid_f64", kind="grid", n=262144, steps=400, h=0.02, a=0.9, nr=801, nth=401,
             node="f64"),
        dict(name="grid_f32_ragged", kind="grid", n=100003, steps=500, h=0.02, a=0.9, nr=401, nth=201,
             node="f32"),
        # a preview image of the benchmark's camera
        dict(name="camera", kind="camera", nx=512, ny=512, a=0.998, incl=math.pi / 3, width=25.0,
             h0=0.1),
        # a training step of the benchmark's adjoint workload
        dict(name="gradient", kind="gradient", n=65536, steps=1024, every=128, h=0.02, a=0.7),
        # initial conditions of a full batch, in both formulations, with their invariants
        dict(name="setup", kind="setup", n=1048576, a=0.9),
    ]


def _log_int(rng, lo, hi):
    """An integer spread evenly over its logarithm, odd and even, round and not."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["orbits", "orbits", "orbits", "monitored", "record", "adaptive", "grid", "grid",
                       "camera", "gradient", "setup"])
    a = round(rng.uniform(0.0, 0.99), 3)
    h = rng.choice([0.01, 0.02])
    form = rng.choice(["christoffel", "christoffel", "hamiltonian"])
    if kind in ("orbits", "monitored"):
        n = _log_int(rng, 64, 1000000)
        steps = _log_int(rng, 10, 2000 if n < 400000 else 900)
        spins = rng.choice([1, 1, 16])
        n = max(spins, n)
        c = dict(kind=kind, n=n, steps=steps, h=h, a=0.99 if spins > 1 else a, spins=spins, ic="bound",
                 form=form, precision=rng.choice(["f64", "f64", "f32k"]), persistent=spins > 1)
        if kind == "monitored":
            c["every"] = _log_int(rng, 10, 1000)
        return c
    if kind == "record":
        every = rng.choice([1, 10, 50])
        return dict(kind=kind, n=_log_int(rng, 64, 200000), steps=every * _log_int(rng, 2, 16),
                    every=every, h=h, a=a, form=form)
    if kind == "adaptive":
        return dict(kind=kind, n=_log_int(rng, 64, 250000), tau=float(rng.choice([50, 200, 400])),
                    tol=rng.choice([1e-12, 1e-11, 1e-10]), a=a)
    if kind == "grid":
        nr = rng.choice([201, 401, 801, rng.randrange(200, 800)])
        return dict(kind=kind, n=_log_int(rng, 64, 250000), steps=_log_int(rng, 10, 400), h=h, a=a,
                    nr=nr, nth=nr // 2 + rng.randrange(0, 2), node=rng.choice(["f64", "f32"]))
    if kind == "camera":
        return dict(kind=kind, nx=_log_int(rng, 16, 500), ny=_log_int(rng, 16, 500),
                    a=rng.choice([0.5, 0.9, 0.998]), incl=round(rng.uniform(0.6, 1.4), 3),
                    width=round(rng.uniform(10.0, 25.0), 2), h0=0.1)
    if kind == "gradient":
        every = rng.choice([32, 64, 128, 256])
        return dict(kind=kind, n=_log_int(rng, 64, 65000), steps=every * _log_int(rng, 1, 1000 // every),
                    every=every, h=h, a=a)
    return dict(kind=kind, n=_log_int(rng, 64, 1000000), a=a)


# ---- inputs ----------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform(g, shape, lo, hi):
    return lo + (hi - lo) * torch.rand(shape, generator=g, dtype=F64, device=DEV)


def _potentials(a, r, s, c, E, L, Q):
    """Carter's radial and polar potentials of a timelike geodesic (M = 1)."""
    P = E * (r * r + a * a) - a * L
    R = P * P - (r * r - 2.0 * r + a * a) * (r * r + (L - a * E) ** 2 + Q)
    T = Q - c * c * (a * a * (1.0 - E * E) + L * L / (s * s))
    return R, T, P


def _carter_velocity(a, r, s, c, E, L, R, T, P, sr, sth):
    rho2 = r * r + a * a * c * c
    delta = r * r - 2.0 * r + a * a
    return torch.stack([((r * r + a * a) * P / delta + a * (L - a * E * s * s)) / rho2,
                        sr * R.clamp(min=0.0).sqrt() / rho2, sth * T.clamp(min=0.0).sqrt() / rho2,
                        (a * P / delta + L / (s * s) - a * E) / rho2])


def _bound(n, a, seed):
    """n random bound orbits: state [8, n] and (E, L_z).  a: a number or a tensor [n]."""
    g = _gen(seed)
    spin = torch.as_tensor(a, dtype=F64, device=DEV).expand(n)
    kept = torch.zeros((7, n), dtype=F64, device=DEV)
    todo = torch.arange(n, device=DEV)
    tries = 16
    while todo.numel():
        k = todo.numel()
        r, th = _uniform(g, (tries, k), *R_RANGE), _uniform(g, (tries, k), *TH_RANGE)
        E, L = _uniform(g, (tries, k), *E_RANGE), _uniform(g, (tries, k), *L_RANGE)
        Q = _uniform(g, (tries, k), *Q_RANGE)
        sign = torch.randint(0, 4, (tries, k), generator=g, device=DEV)
        R, T, _ = _potentials(spin[todo], r, th.sin(), th.cos(), E, L, Q)
        ok = (R >= 0.0) & (T >= 0.0)
        first = ok.to(torch.uint8).argmax(dim=0, keepdim=True)
        hit = ok.any(dim=0)
        rows = torch.stack([x.gather(0, first)[0] for x in
                            (r, th, E, L, Q, 1.0 - 2.0 * (sign & 1).to(F64), 1.0 - (sign & 2).to(F64))])
        kept[:, todo[hit]] = rows[:, hit]
        todo = todo[~hit]
    r, th, E, L, Q, sr, sth = kept
    s, c = th.sin(), th.cos()
    R, T, P = _potentials(spin, r, s, c, E, L, Q)
    state = torch.zeros((8, n), dtype=F64, device=DEV)
    state[1], state[2] = r, th
    state[4:] = _carter_velocity(spin, r, s, c, E, L, R, T, P, sr, sth)
    return state, E, L


def _circular(n, seed):
    """n near-circular equatorial Schwarzschild orbits, L off by up to 1e-3."""
    g = _gen(seed)
    r = _uniform(g, (n,), 6.5, 20.0)
    L = r / (r - 3.0).sqrt() * (1.0 + _uniform(g, (n,), -1e-3, 1e-3))
    f = 1.0 - 2.0 / r
    state = torch.zeros((8, n), dtype=F64, device=DEV)
    state[1], state[2] = r, 0.5 * math.pi
    state[4] = ((1.0 + L * L / (r * r)) / f).sqrt()
    state[7] = L / (r * r)
    return state


def _spins(case):
    """The batch's spacetimes and each lane's index into them (None for one spacetime)."""
    k = case.get("spins", 1)
    if k == 1:
        return [(1.0, case["a"])], None
    lanes = torch.arange(case["n"], device=DEV, dtype=torch.int64) * k // case["n"]
    return [(1.0, case["a"] * j / (k - 1)) for j in range(k)], lanes.to(torch.int32)


def _spin_of_lane(case):
    st, lanes = _spins(case)
    return st[0][1] if lanes is None else torch.tensor([x[1] for x in st], dtype=F64, device=DEV)[lanes.long()]


def _start(case, seed):
    a = _spin_of_lane(case)
    state = _circular(case["n"], seed) if case.get("ic") == "circular" else _bound(case["n"], a, seed)[0]
    if case.get("form") == "hamiltonian" or case["kind"] == "grid":
        state[4:] = _lower(a, state)
    return state


def _grid_nodes(case):
    """The five 3+1 functions of Kerr on the case's grid, as a caller's own metric."""
    nr, nth, a = case["nr"], case["nth"], case["a"]
    r0, dr = 1.5 if a > 0.87 else 2.1, 60.0 / (nr - 1)
    th0, dth = 0.1, (math.pi - 0.2) / (nth - 1)
    r = (r0 + dr * torch.arange(nr, dtype=F64, device=DEV))[:, None]
    th = (th0 + dth * torch.arange(nth, dtype=F64, device=DEV))[None, :]
    rho2 = r * r + (a * th.cos()) ** 2
    delta = r * r - 2.0 * r + a * a
    sigma = (r * r + a * a) ** 2 - a * a * delta * th.sin() ** 2
    nodes = torch.stack([(rho2 * delta / sigma).sqrt(), -2.0 * a * r / sigma, rho2 / delta,
                         rho2.expand_as(sigma), sigma / rho2], dim=-1).contiguous()
    nodes = nodes.to(torch.float32) if case["node"] == "f32" else nodes
    r_stop = max(1.2 * (1.0 + math.sqrt(1.0 - a * a)), r0 + 2.0 * dr)
    return nodes, r0, dr, th0, dth, r_stop


def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    if kind == "camera":
        # another seed: another place of the camera, within a tenth of a degree
        s["cam"] = m.Camera(a=case["a"], incl=_incl(case, seed), half_width=case["width"], nx=case["nx"],
                            ny=case["ny"], h0=case["h0"])
        return s
    if kind == "setup":
        s["spec"] = m.ICSpec(mode=m.IC_CONSTANTS, seed=int(seed))
        return s
    if kind == "gradient":
        p, s["E"], s["target"] = _params(case, seed)
        s["p"] = p.requires_grad_(True)
        return s
    s["start"] = _start(case, seed)
    s["st"], s["lanes"] = _spins(case)
    if kind == "grid":
        nodes, r0, dr, th0, dth, r_stop = _grid_nodes(case)
        s["grid"] = m.Grid(nodes, r0, dr, th0, dth, r_stop)
    if case.get("persistent"):
        s["ws"] = torch.empty(m.workspace_bytes(m.OP_INTEGRATE, case["n"], 1), dtype=torch.uint8, device=DEV)
    return s


def _incl(case, seed):
    return case["incl"] + 1e-3 * (int(seed) % 1009) / 1009.0


def _params(case, seed):
    """Parameters (r0, theta0, u^r0, u^theta0, L_z) and E of bound orbits, and a target."""
    y, E, L = _bound(case["n"], case["a"], seed)
    target = torch.stack([y[1], y[2], torch.zeros_like(E)]) + 0.5
    return torch.stack([y[1], y[2], y[5], y[6], L]).contiguous(), E, target


# ---- one pass --------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "camera":
        return m.trace_camera(s["cam"])
    if kind == "setup":
        st = [(1.0, case["a"])]
        state, consts, attempts = m.init_particles(s["spec"], st, case["n"])
        inv = m.invariants(state, st)
        momenta = m.convert_state(state.clone(), st, True)
        return {"state": state, "consts": consts, "attempts": attempts, "invariants": inv,
                "momenta": momenta}
    if kind == "gradient":
        y, status, steps = m.IntegrateFromParams.apply(s["p"], s["E"], (1.0, case["a"]), case["h"],
                                                       case["steps"], case["every"])
        loss = ((y[1:4] - s["target"]) ** 2).sum()
        grad, = torch.autograd.grad(loss, s["p"])
        return {"state": y.detach(), "status": status, "steps": steps, "grad": grad}
    state = s["start"].clone()
    status, steps = m.new_lane_arrays(case["n"])
    out = {"state": state, "status": status, "steps": steps}
    if kind == "orbits":
        m.integrate(state, status, steps, s["st"], h=case["h"], n_steps=case["steps"],
                    precision=case["precision"], formulation=case["form"], st_of_lane=s["lanes"],
                    persistent=case["persistent"], ws=s.get("ws"))
    elif kind == "monitored":
        out["monitor"] = m.integrate_monitored(state, status, steps, s["st"], case["h"], case["steps"],
                                               case["every"], precision=case["precision"],
                                               formulation=case["form"], st_of_lane=s["lanes"],
                                               persistent=case["persistent"], ws=s.get("ws"))
    elif kind == "record":
        out["records"] = m.integrate_record(state, status, steps, s["st"], case["h"], case["steps"],
                                            case["every"], formulation=case["form"])
    elif kind == "grid":
        m.integrate_grid(state, status, steps, s["grid"], case["h"], case["steps"], 55.0)
    else:
        tau = torch.zeros(case["n"], dtype=F64, device=DEV)
        h = torch.full((case["n"],), 0.1, dtype=F64, device=DEV)
        rejects = torch.zeros(case["n"], dtype=torch.int32, device=DEV)
        m.integrate_adaptive(state, tau, h, status, steps, rejects, s["st"], case["tau"],
                             rtol=case["tol"], atol=case["tol"])
        out.update(tau=tau, h=h, rejects=rejects)
    return out


# ---- what a pass cannot do without -------------------------------------------------------
def work(case):
    """Bytes: each input read once and each output written once.  Operations: those of the
    right-hand sides and Runge-Kutta sums (a multiply-add is two); the adaptive attempts and
    the camera's steps, which depend on the lane, by their usual number."""
    kind = case["kind"]
    n = case.get("n", 0) or case["nx"] * case["ny"]
    lane = 64 + 64 + 8 + 8  # state in and out, status and steps in and out
    per_step = {("f64", "christoffel"): 514, ("f64", "hamiltonian"): 336,
                ("f32k", "christoffel"): 562, ("f32k", "hamiltonian"): 386}
    if kind in ("orbits", "monitored", "record"):
        b = lane + (128 if kind == "monitored" else 40 * (case["steps"] // case["every"]) if kind == "record" else 0)
        return {"bytes": n * b, "flops": n * case["steps"] * per_step[case.get("precision", "f64"), case["form"]]}
    if kind == "adaptive":
        return {"bytes": n * (lane + 32 + 8), "flops": n * 1024 * 0.44 * case["tau"] * (1e-10 / case["tol"]) ** 0.2}
    if kind == "grid":
        nodes = case["nr"] * case["nth"] * 5 * (8 if case["node"] == "f64" else 4)
        return {"bytes": n * lane + nodes, "flops": n * case["steps"] * (4 * (440 + 130) + 80)}
    if kind == "camera":
        return {"bytes": n * 24, "flops": n * 640 * 514}
    if kind == "gradient":
        slots = case["steps"] // case["every"] + 1
        return {"bytes": n * (6 * 8 + 64 + 8 + 40 + 2 * 64 * slots), "flops": n * case["steps"] * 514 * 5}
    return {"bytes": n * (64 + 32 + 8 + 64 + 32 + 128), "flops": n * 20 * 100}


# ---- the same in plain double precision --------------------------------------------------
def _metric(a, r, th):
    s2, c2 = th.sin() ** 2, th.cos() ** 2
    rho2, delta = r * r + a * a * c2, r * r - 2.0 * r + a * a
    q = 2.0 * r / rho2
    return q - 1.0, -a * q * s2, (r * r + a * a + a * a * q * s2) * s2, rho2 / delta, rho2


def _lower(a, y):
    tt, tp, pp, rr, hh = _metric(a, y[1], y[2])
    return torch.stack([tt * y[4] + tp * y[7], rr * y[5], hh * y[6], tp * y[4] + pp * y[7]])


def _invariants(a, y):
    p = _lower(a, y)
    norm = (p * y[4:]).sum(dim=0)
    s2, c2 = y[2].sin() ** 2, y[2].cos() ** 2
    return torch.stack([-p[0], p[3], p[2] ** 2 + c2 * (a * a * (-norm - p[0] ** 2) + p[3] ** 2 / s2), norm])


def _christoffel(a, y):
    """d(x, u)/dtau of Kerr, M = 1: the lowered geodesic equation, raised."""
    _, r, th, _, ut, ur, uh, up = y
    s, c = th.sin(), th.cos()
    s2, sc, a2 = s * s, s * c, a * a
    rho2, delta, A = r * r + a2 * c * c, r * r - 2.0 * r + a2, r * r + a2
    q = 2.0 * r / rho2
    q_r, q_h = (2.0 - 2.0 * r * q) / rho2, 2.0 * q * a2 * sc / rho2
    tt_r, tt_h = q_r, q_h
    tp_r, tp_h = -a * q_r * s2, -a * (q_h * s2 + 2.0 * q * sc)
    pp_r = (2.0 * r + a2 * q_r * s2) * s2
    pp_h = a2 * (q_h * s2 + 2.0 * q * sc) * s2 + 2.0 * (A + a2 * q * s2) * sc
    rr = rho2 / delta
    rr_r, rr_h = (2.0 * r - rr * (2.0 * r - 2.0)) / delta, -2.0 * a2 * sc / delta
    hh_r, hh_h = 2.0 * r, -2.0 * a2 * sc
    Dt, Dp = ur * tt_r + uh * tt_h, ur * tp_r + uh * tp_h
    Ft = -(Dt * ut + Dp * up)
    Fp = -(Dp * ut + (ur * pp_r + uh * pp_h) * up)
    Fr = 0.5 * (tt_r * ut * ut + 2.0 * tp_r * ut * up + pp_r * up * up + hh_r * uh * uh - rr_r * ur * ur) - rr_h * ur * uh
    Fh = 0.5 * (tt_h * ut * ut + 2.0 * tp_h * ut * up + pp_h * up * up + rr_h * ur * ur - hh_h * uh * uh) - hh_r * ur * uh
    gtt, gtp, gpp = q - 1.0, -a * q * s2, (A + a2 * q * s2) * s2
    det = -delta * s2
    return torch.stack([ut, ur, uh, up, (gpp * Ft - gtp * Fp) / det, Fr / rr, Fh / rho2,
                        (gtt * Fp - gtp * Ft) / det])


def _canonical(a, z):
    """d(x, p)/dtau: Hamilton's equations of the separated Kerr Hamiltonian, M = 1."""
    _, r, th, _, pt, pr, ph, pp = z
    s, c = th.sin(), th.cos()
    A, rho2, delta = r * r + a * a, r * r + a * a * c * c, r * r - 2.0 * r + a * a
    P, w = A * pt + a * pp, pp / s + a * s * pt
    N = delta * pr * pr + ph * ph + w * w - P * P / delta
    N_r = 2.0 * ((r - 1.0) * pr * pr - P / delta * (2.0 * r * pt - P / delta * (r - 1.0)))
    N_h = 2.0 * w * c * (a * pt - pp / (s * s))
    zero = torch.zeros_like(r)
    return torch.stack([(a * s * w - A * P / delta) / rho2, delta * pr / rho2, ph / rho2,
                        (w / s - a * P / delta) / rho2, zero, (r * N / rho2 - 0.5 * N_r) / rho2,
                        -(a * a * s * c * N / rho2 + 0.5 * N_h) / rho2, zero])


def _lagrange(u):
    w = [-u * (u - 1.0) * (u - 2.0) / 6.0, (u + 1.0) * (u - 1.0) * (u - 2.0) / 2.0,
         -(u + 1.0) * u * (u - 2.0) / 2.0, (u + 1.0) * u * (u - 1.0) / 6.0]
    d = [-(3.0 * u * u - 6.0 * u + 2.0) / 6.0, (3.0 * u * u - 4.0 * u - 1.0) / 2.0,
         -(3.0 * u * u - 2.0 * u - 2.0) / 2.0, (3.0 * u * u - 1.0) / 6.0]
    return torch.stack(w), torch.stack(d)


def _gridded(grid, z):
    """Hamilton's equations in the metric that 4-point Lagrange interpolation makes of the nodes."""
    nodes, r0, dr, th0, dth, _ = grid
    nr, nth, _ = nodes.shape
    _, r, th, _, pt, pr, ph, pp = z
    x, t = (r - r0) / dr, (th - th0) / dth
    i = x.nan_to_num(1.0).floor().clamp(1, nr - 3)
    j = t.nan_to_num(1.0).floor().clamp(1, nth - 3)
    (wr, dr_), (wt, dt_) = _lagrange(x - i), _lagrange(t - j)
    at = ((i.long() - 1) * nth + (j.long() - 1))[None, None] + \
        (torch.arange(4, device=DEV)[:, None] * nth + torch.arange(4, device=DEV)[None, :])[:, :, None]
    f = nodes.reshape(-1, 5)[at].to(F64)  # [4, 4, n, 5]
    rows, rows_t = (f * wt[None, :, :, None]).sum(1), (f * dt_[None, :, :, None]).sum(1)
    F = (rows * wr[:, :, None]).sum(0).unbind(-1)
    Fr = ((rows * dr_[:, :, None]).sum(0) / dr).unbind(-1)
    Ft = ((rows_t * wr[:, :, None]).sum(0) / dth).unbind(-1)
    s, c = th.sin(), th.cos()
    al, be, grr, ghh, gpp = F[0], F[1], F[2], F[3], F[4] * s * s
    ut = (be * pp - pt) / (al * al)
    ur, uh, w = pr / grr, ph / ghh, pp / gpp

    def force(D, dgpp):  # (1/2) (d_l g_ab) u^a u^b
        return -al * D[0] * ut * ut + pp * D[1] * ut + 0.5 * (D[2] * ur * ur + D[3] * uh * uh + dgpp * w * w)

    zero = torch.zeros_like(r)
    return torch.stack([ut, ur, uh, w - be * ut, zero, force(Fr, Fr[4] * s * s),
                        force(Ft, Ft[4] * s * s + 2.0 * F[4] * s * c), zero])


def _rk4(f, h, y):
    k1 = f(y)
    y2 = y + 0.5 * h * k1
    k2 = f(y2)
    y3 = y + 0.5 * h * k2
    k3 = f(y3)
    y4 = y + h * k3
    return y + h / 6.0 * (k1 + 2.0 * (k2 + k3) + f(y4)), torch.stack([y2[1:3], y3[1:3], y4[1:3]])


def _usable(y):
    return y.isfinite().all(dim=0) & (y[2] > 0.0) & (y[2] < math.pi)


def _r_stop(a):
    a = torch.as_tensor(a, dtype=F64, device=DEV)
    return HORIZON_FACTOR * (1.0 + (1.0 - a * a).sqrt())


def _fixed(f, case, y, r_stop, grid=None, each=None):
    """Fixed-step RK4 of all lanes with the stop rules; each(k, y, taken) sees the state after
    step k and the steps that each lane has evaluated."""
    live = torch.ones(y.shape[1], dtype=torch.bool, device=DEV)
    taken = torch.zeros(y.shape[1], dtype=F64, device=DEV)
    resc = 55.0 if grid else R_ESCAPE
    for k in range(case["steps"]):
        taken += live
        y1, pts = _rk4(f, case["h"], y)
        keep = live & (pts[:, 0] > r_stop).all(dim=0) & _usable(y1)
        if grid:
            nodes, r0, dr, th0, dth, _ = grid
            q = torch.cat([pts, y1[None, 1:3]])
            keep &= ((q[:, 0] >= r0 + dr) & (q[:, 0] <= r0 + (nodes.shape[0] - 2) * dr)
                     & (q[:, 1] >= th0 + dth) & (q[:, 1] <= th0 + (nodes.shape[1] - 2) * dth)).all(dim=0)
        y = torch.where(keep, y1, y)
        live = keep & (y[1] > r_stop) & (y[1] < resc)
        if each:
            each(k, y, taken)
    return y


# Dormand and Prince, 5(4)
_DP_A = [[1 / 5], [3 / 40, 9 / 40], [44 / 45, -56 / 15, 32 / 9],
         [19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729],
         [9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656],
         [35 / 384, 0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84]]
_DP_E = [71 / 57600, 0, -71 / 16695, 71 / 1920, -17253 / 339200, 22 / 525, -1 / 40]


def _adaptive(f, y, tau_end, tol, r_stop):
    n = y.shape[1]
    tau = torch.zeros(n, dtype=F64, device=DEV)
    h = torch.full((n,), 0.1, dtype=F64, device=DEV)
    capped = torch.zeros(n, dtype=torch.bool, device=DEV)
    lanes, out, tau_out = torch.arange(n, device=DEV), y.clone(), tau.clone()
    k1 = f(y)
    while lanes.numel():
        last = tau + h >= tau_end
        hh = torch.where(last, tau_end - tau, h)
        ks, ok = [k1], torch.ones_like(last)
        for row in _DP_A:
            p = y + hh * sum(b * k for b, k in zip(row, ks) if b)
            if len(ks) < 6:
                ok = ok & (p[1] > r_stop)
            ks.append(f(p))
        e = hh * sum(b * k for b, k in zip(_DP_E, ks) if b)
        err = (e / (tol + tol * torch.maximum(y.abs(), p.abs()))).square().mean(dim=0).sqrt()
        ok = ok & _usable(p) & err.isfinite()
        grow = (0.9 * err.clamp(min=1e-300) ** -0.2).clamp(min=0.2)
        accept = ok & (err <= 1.0)
        h = torch.where(accept, hh * torch.where(capped, grow.clamp(max=1.0), grow.clamp(max=5.0)),
                        hh * grow.clamp(max=1.0))
        capped = ~accept
        y, k1 = torch.where(accept, p, y), torch.where(accept, ks[6], k1)
        tau = torch.where(accept, torch.where(last, torch.full_like(tau, tau_end), tau + hh), tau)
        done = ~ok | (accept & ((y[1] <= r_stop) | (y[1] >= R_ESCAPE) | (tau >= tau_end)))
        out[:, lanes[done]], tau_out[lanes[done]] = y[:, done], tau[done]
        if done.any():
            go = ~done
            lanes, y, k1, tau, h, capped = lanes[go], y[:, go], k1[:, go], tau[go], h[go], capped[go]
    return out, tau_out


def _image(case, seed):
    """(r_c, phi_c) of the disk crossings of all rays, NaN elsewhere."""
    a, i, w, nx, ny = case["a"], _incl(case, seed), case["width"], case["nx"], case["ny"]
    p = torch.arange(nx * ny, device=DEV)
    alpha = -w + ((p % nx).to(F64) + 0.5) * 2.0 * w / nx
    beta = -w + ((p // nx).to(F64) + 0.5) * 2.0 * w / ny
    s, c, r = math.sin(i), math.cos(i), 1000.0
    L, Q = -alpha * s, beta * beta + c * c * (alpha * alpha - a * a)
    P = (r * r + a * a) - a * L
    delta, rho2 = r * r - 2.0 * r + a * a, r * r + a * a * c * c
    R = P * P - delta * ((L - a) ** 2 + Q)
    T = Q - c * c * (L * L / (s * s) - a * a)
    u = [((r * r + a * a) * P / delta + a * (L - a * s * s)) / rho2, R.clamp(min=0.0).sqrt() / rho2,
         torch.where(beta >= 0.0, 1.0, -1.0) * T.clamp(min=0.0).sqrt() / rho2,
         (a * P / delta + L / (s * s) - a) / rho2]
    y = torch.stack([torch.zeros_like(P), torch.full_like(P, r), torch.full_like(P, i), torch.zeros_like(P)]
                    + [-x for x in u])
    z1 = 1.0 + (1.0 - a * a) ** (1 / 3) * ((1.0 + a) ** (1 / 3) + (1.0 - a) ** (1 / 3))
    z2 = math.sqrt(3.0 * a * a + z1 * z1)
    r_in = 3.0 + z2 - math.sqrt((3.0 - z1) * (3.0 + z1 + 2.0 * z2))
    stop, hit = _r_stop(a), torch.full((2, nx * ny), math.nan, dtype=F64, device=DEV)
    k = 0
    while p.numel() and k < 100000:
        y1, pts = _rk4(lambda v: _christoffel(a, v), case["h0"] * (y[1] / 10.0).clamp(min=1.0), y)
        good = (pts[:, 0] > stop).all(dim=0) & _usable(y1)
        cross = good & ((y[2] > 0.5 * math.pi) != (y1[2] > 0.5 * math.pi))
        c0, c1 = y[2].cos(), y1[2].cos()
        f = c0 / (c0 - c1)
        rc, pc = y[1] + (y1[1] - y[1]) * f, y[3] + (y1[3] - y[3]) * f
        disk = cross & (rc >= r_in) & (rc <= 30.0)
        hit[0, p[disk]], hit[1, p[disk]] = rc[disk], pc[disk]
        go = good & ~disk & (y1[1] > stop) & (y1[1] < R_ESCAPE)
        k += 1
        if k % 16 == 0:  # drop the finished rays now and then, park them in between
            p, y = p[go], y1[:, go]
        else:
            y = torch.where(go, y1, torch.full_like(y1, math.nan))
    return hit


def _orbit_from_params(p, E, a):
    r, th, ur, uh, L = p
    s2, c2 = th.sin() ** 2, th.cos() ** 2
    rho2, delta = r * r + a * a * c2, r * r - 2.0 * r + a * a
    sigma = (r * r + a * a) ** 2 - a * a * delta * s2
    den, zero = rho2 * delta, torch.zeros_like(r)
    return torch.stack([zero, r, th, zero, (sigma * E - 2.0 * a * r * L) / den, ur, uh,
                        (2.0 * a * r * E + (delta - a * a * s2) / s2 * L) / den])


def _gradient(case, seed):
    p, E, target = _params(case, seed)
    a, h = case["a"], case["h"]
    stop = _r_stop(a)
    f = lambda v: _christoffel(a, v)  # noqa: E731
    p.requires_grad_(True)
    y0 = _orbit_from_params(p, E, a)
    y, live = y0.detach(), torch.ones(case["n"], dtype=torch.bool, device=DEV)
    kept = []
    for _ in range(case["steps"]):
        y1, pts = _rk4(f, h, y)
        keep = live & (pts[:, 0] > stop).all(dim=0) & _usable(y1)
        kept.append((y, keep))
        y = torch.where(keep, y1, y)
        live = keep & (y[1] > stop) & (y[1] < R_ESCAPE)
    lam = torch.zeros_like(y)
    lam[1:4] = 2.0 * (y[1:4] - target)
    for x, keep in reversed(kept):
        x = x.clone().requires_grad_(True)
        g, = torch.autograd.grad(_rk4(f, h, x)[0], x, lam)
        lam = torch.where(keep, g, lam)
    grad, = torch.autograd.grad(y0, p, lam)
    return {"state": y, "status": None, "steps": None, "grad": grad}


def _splitmix(seed, index):
    """Outputs of the SplitMix64 sequence at the given indices (int64 arithmetic mod 2^64)."""
    def signed(v):
        return v - (1 << 64) if v >= 1 << 63 else v

    def shift(x, k):  # logical
        return (x >> k) & ((1 << (64 - k)) - 1)
    z = int(seed) + (index + 1) * signed(0x9E3779B97F4A7C15)
    z = (z ^ shift(z, 30)) * signed(0xBF58476D1CE4E5B9)
    z = (z ^ shift(z, 27)) * signed(0x94D049BB133111EB)
    return z ^ shift(z, 31)


def _setup(case, seed):
    a, n = case["a"], case["n"]
    found = torch.zeros((7, n), dtype=F64, device=DEV)
    todo, attempt = torch.arange(n, device=DEV), 0
    ranges = (R_RANGE, TH_RANGE, E_RANGE, L_RANGE, Q_RANGE)
    while todo.numel():
        x = [_splitmix(seed, (todo << 24) | (attempt << 4) | k) for k in range(7)]
        v = [lo + (hi - lo) * (((u >> 11) & ((1 << 53) - 1)).to(F64) * 2.0 ** -53)
             for (lo, hi), u in zip(ranges, x)]
        v += [1.0 - 2.0 * (u < 0).to(F64) for u in x[5:]]
        R, T, _ = _potentials(a, v[0], v[1].sin(), v[1].cos(), v[2], v[3], v[4])
        ok = (R >= 0.0) & (T >= 0.0)
        found[:, todo[ok]] = torch.stack(v)[:, ok]
        todo, attempt = todo[~ok], attempt + 1
    r, th, E, L, Q, sr, sth = found
    s, c = th.sin(), th.cos()
    R, T, P = _potentials(a, r, s, c, E, L, Q)
    state = torch.zeros((8, n), dtype=F64, device=DEV)
    state[1], state[2] = r, th
    state[4:] = _carter_velocity(a, r, s, c, E, L, R, T, P, sr, sth)
    momenta = state.clone()
    momenta[4:] = _lower(a, state)
    return {"state": state, "consts": torch.stack([E, L, Q, torch.ones_like(E)]), "attempts": None,
            "invariants": _invariants(a, state), "momenta": momenta}


def exact(case, seed):
    kind = case["kind"]
    if kind == "camera":
        return {"status": None, "steps": None, "hit": _image(case, seed)}
    if kind == "setup":
        return _setup(case, seed)
    if kind == "gradient":
        return _gradient(case, seed)
    a = _spin_of_lane(case)
    y = _start(case, seed)
    if kind == "adaptive":
        state, tau = _adaptive(lambda v: _christoffel(a, v), y, case["tau"], case["tol"], _r_stop(a))
        # the next step size h follows the rounding of the error estimate
        return {"state": state, "status": None, "steps": None, "tau": tau, "h": None, "rejects": None}
    if kind == "grid":
        grid = _grid_nodes(case)
        y = _fixed(lambda v: _gridded(grid, v), case, y, grid[5], grid=grid)
        return {"state": y, "status": None, "steps": None}
    rhs = _canonical if case["form"] == "hamiltonian" else _christoffel
    out = {"status": None, "steps": None}
    if kind == "monitored":
        out["monitor"] = None  # running maxima of differences that are mostly rounding
    records = []

    def record(k, v, taken):
        if (k + 1) % case["every"] == 0:
            rr = (v[1] ** 2 + a * a).sqrt()
            records.append(torch.stack([case["h"] * taken, v[0], rr * v[2].sin() * v[3].cos(),
                                        rr * v[2].sin() * v[3].sin(), v[1] * v[2].cos()]))
    out["state"] = _fixed(lambda v: rhs(a, v), case, y, _r_stop(a),
                          each=record if kind == "record" else None)
    if kind == "record":
        out["records"] = torch.stack(records)
    return out
