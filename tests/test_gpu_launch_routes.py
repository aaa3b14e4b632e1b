"""The launch routes that a default shape can take (in turns, the idle queue left to one thread per
lane, spans between monitored steps, several launches in turns) under hipGraph capture and on two
streams at once: the bits of the plain launch on the default stream."""
import math

import pytest

pytestmark = pytest.mark.gpu

KERR = [(1.0, 0.9)]
SPINS = [(1.0, 0.99 * k / 15) for k in range(16)]


def states(m, n, sts, seed, ham=False):
    import torch
    sol = torch.arange(n, dtype=torch.int32, device="cuda") % len(sts) if len(sts) > 1 else None
    s, _, _ = m.init_particles(m.ICSpec(mode=m.IC_CONSTANTS, seed=seed), sts, n, st_of_lane=sol)
    s[5, ::97] = -30.0
    if ham:
        m.convert_state(s, sts, True, st_of_lane=sol)
    return s, sol


def orbits(m, seed, n, steps=100, sts=KERR, plain=None, monitor=0, **kw):
    """(buffers, run, run in the plain shape)"""
    import torch
    s0, sol = states(m, n, sts, seed, kw.get("formulation") == "hamiltonian")
    bufs = [torch.empty_like(s0), *m.new_lane_arrays(n)]
    if monitor:
        bufs.append(torch.empty((8, n), dtype=torch.float64, device="cuda"))
    ws = torch.empty(256, dtype=torch.uint8, device="cuda") if kw.get("persistent") else None

    def run(**shape):
        bufs[0].copy_(s0)
        bufs[1].zero_()
        bufs[2].zero_()
        a = dict(kw, h=0.02, n_steps=steps, st_of_lane=sol, ws=ws, **shape)
        if monitor:
            m.integrate_monitored(*bufs[:3], sts, monitor_every=monitor, monitor=bufs[3], **a)
        else:
            m.integrate(*bufs[:3], sts, **a)
    return bufs, run, lambda: run(**plain)


def records(m, seed, n):
    import torch
    s0, _ = states(m, n, KERR, seed)
    bufs = [torch.empty_like(s0), *m.new_lane_arrays(n),
            torch.empty((7, 5, n), dtype=torch.float64, device="cuda")]

    def run(**shape):
        bufs[0].copy_(s0)
        bufs[1].zero_()
        bufs[2].zero_()
        m.integrate_record(*bufs[:3], KERR, 0.02, 140, 20, traj=bufs[3], **shape)
    return bufs, run, lambda: run(block=256)


def gridded(m, seed, n, steps=100, **kw):
    import torch
    g = m.grid_kerr(1.0, 0.9, 401, 201, 1.5, 60.0 / 400, 0.1, (math.pi - 0.2) / 200, 1.72)
    s0, _ = states(m, n, KERR, seed, True)
    bufs = [torch.empty_like(s0), *m.new_lane_arrays(n)]

    def run(**shape):
        bufs[0].copy_(s0)
        bufs[1].zero_()
        bufs[2].zero_()
        m.integrate_grid(*bufs, g, 0.02, steps, 55.0, **kw, **shape)
    return bufs, run, lambda: run(block=256)


def image(m, seed, n):
    import torch
    cam = dict(a=0.998, nx=n, ny=n, half_width=20.0 + seed)
    out = m.trace_camera(m.Camera(**cam, persistent=0))
    bufs = list(out.values())
    ws = torch.empty(m.workspace_bytes(m.OP_CAMERA, n * n), dtype=torch.uint8, device="cuda")
    for v in bufs:
        v.zero_()

    def run(**shape):
        m.trace_camera(m.Camera(**cam, **shape), out=out, ws=ws)
    return bufs, run, lambda: run(persistent=0)


ROUTES = {
    "turns": lambda m, s: orbits(m, s, 65536 + 3000, plain=dict(block=256)),
    "turns, hamiltonian": lambda m, s: orbits(m, s, 300007, formulation="hamiltonian", plain=dict(block=256)),
    "turns, 16 spacetimes": lambda m, s: orbits(m, s, 131072 + 5000, sts=SPINS, plain=dict(block=256)),
    "turns, several launches": lambda m, s: orbits(m, s, 65536 + 3000, steps=250, steps_per_chunk=100,
                                                   plain=dict(block=256)),
    "records in turns": lambda m, s: records(m, s, 100003),
    "gridded in turns": lambda m, s: gridded(m, s, 131072 + 5000),
    "gridded in turns, several launches": lambda m, s: gridded(m, s, 65536 + 3000, steps=250, steps_per_chunk=100),
    "idle queue": lambda m, s: orbits(m, s, 20000, sts=SPINS, persistent=True, plain=dict(steps_per_chunk=64)),
    "idle queue in turns": lambda m, s: orbits(m, s, 65536 + 3000, persistent=True, plain=dict(steps_per_chunk=64)),
    "idle queue, f32k": lambda m, s: orbits(m, s, 20000, sts=SPINS, persistent=True, precision="f32k",
                                            plain=dict(steps_per_chunk=64)),
    "spans, f32k": lambda m, s: orbits(m, s, 20000, precision="f32k", monitor=25,
                                       plain=dict(persistent=True, steps_per_chunk=1)),
    "idle queue, monitored": lambda m, s: orbits(m, s, 20000, sts=SPINS, persistent=True, monitor=25,
                                                 plain=dict(steps_per_chunk=64)),
    "camera": lambda m, s: image(m, s, 96),
}



@pytest.mark.parametrize("route", ROUTES)
def test_route_under_capture(route):
    """Three replays, with the buffers spoilt and eager work between them."""
    import torch

    import paper_1803_08320_amd as m
    bufs, run, plain = ROUTES[route](m, 5)
    plain()
    torch.cuda.synchronize()
    want = [x.clone() for x in bufs]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        run()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run()
    for rep in range(3):
        for x in bufs:
            x.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for k, (x, y) in enumerate(zip(bufs, want)):
            assert torch.equal(torch.nan_to_num(x), torch.nan_to_num(y)), (rep, k)
        run()  # eager work between replays
        torch.cuda.synchronize()
        for k, (x, y) in enumerate(zip(bufs, want)):
            assert torch.equal(torch.nan_to_num(x), torch.nan_to_num(y)), (rep, k)


@pytest.mark.parametrize("route", ROUTES)
def test_route_on_two_streams(route):
    """Two batches at once, each on a stream of its own, several times."""
    import torch

    import paper_1803_08320_amd as m
    jobs = [ROUTES[route](m, seed) for seed in (5, 6)]
    want = []
    for bufs, run, plain in jobs:
        plain()
        torch.cuda.synchronize()
        want.append([x.clone() for x in bufs])
    streams = [torch.cuda.Stream() for _ in jobs]
    for rep in range(3):
        for x in (x for bufs, _, _ in jobs for x in bufs):
            x.fill_(-1)
        torch.cuda.synchronize()
        for s, (bufs, run, _) in zip(streams, jobs):
            with torch.cuda.stream(s):
                run()
        torch.cuda.synchronize()
        for w, (bufs, _, _) in zip(want, jobs):
            for k, (x, y) in enumerate(zip(bufs, w)):
                assert torch.equal(torch.nan_to_num(x), torch.nan_to_num(y)), (rep, k)
