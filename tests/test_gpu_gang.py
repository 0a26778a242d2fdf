"""The resident gang behind pso_run: every instantiation at the edges of its
shapes (one part and many, particles past the last part's, dimensions past the
last chunk's, two to sixteen lanes per particle), bit for bit against the
oracle -- state, history, improvement count, continued runs, stop rule --;
parameters at the limits of what it accepts; and gangs that cannot all be
resident together."""
import threading

import numpy as np
import pytest

import paper_2205_01313_amd as pso
from paper_2205_01313_amd import workloads as wl
from tests.gpu_util import announce, assert_state_equal, gpu_swarm, oracle_swarm

pytestmark = pytest.mark.gpu


def run_parts(g, cuts, tol=0.0, f_star=0.0):
    r = None
    for n in cuts:
        r = g.run(n, tol=tol, f_star=f_star)
    return r


def check(spec, cuts, tol=0.0, f_star=0.0):
    T = sum(cuts)
    with gpu_swarm(spec) as g:
        r = run_parts(g, cuts, tol, f_star)
        st = g.state()
        hist = g.history(0, st["t"] + 1)
        imp = g.counters()["pbest_improvements"]
    o = oracle_swarm(spec, 8).run_f32(T, tol=tol, f_star=f_star)
    assert st["t"] == o["iters"] and r["gbest_fit"] == o["gbest_fit"] and r["gbest_iter"] == o["giter"]
    assert np.array_equal(hist, o["hist"])
    assert_state_equal(st, o, spec.N, spec.D)
    return imp, st, hist


# "C,P": dimensions of a lane, particles of a part
@pytest.mark.parametrize("fit,N,D,shape", [
    ("sphere", 1, 1, "2,64"), ("cubic", 65, 1, "2,64"), ("rastrigin", 1000, 2, "2,256"), ("ackley", 4001, 2, "2,1024"),
    ("rosenbrock", 257, 3, "4,256"), ("sphere", 700, 7, "8,512"), ("cubic", 1025, 8, "8,1024"),
    ("rastrigin", 900, 13, "16,512"), ("ackley", 1500, 16, "16,1024"), ("rosenbrock", 1100, 31, "32,1024"),
    ("sphere", 600, 63, "64,512"), ("rastrigin", 130, 3, "2,64"), ("rosenbrock", 200, 9, "2,128"),
    ("ackley", 321, 17, "4,64"), ("rosenbrock", 500, 33, "8,64"), ("cubic", 64, 65, "8,64"),
    ("rastrigin", 129, 47, "16,128"), ("rosenbrock", 70, 18, "16,64"), ("sphere", 33, 31, "2,16"),
    ("rosenbrock", 50, 21, "2,32"), ("ackley", 95, 13, "4,32"), ("rastrigin", 40, 101, "8,16"),
    ("rosenbrock", 47, 70, "8,32"), ("rosenbrock", 150, 19, "4,152"), ("ackley", 71, 49, "8,72"), ("cubic", 77, 1, "1,64"), ("rosenbrock", 300, 127, "64,256"), ("ackley", 300, 66, "64,256"),
    ("cubic", 130, 129, "64,64"), ("rastrigin", 129, 125, "64,128")])
def test_gang_shapes_equal_oracle(monkeypatch, fit, N, D, shape):
    spec = wl.SwarmSpec(fit, N, D, 60, seed=N * 3 + D, shift_amplitude=1.5)
    announce(f"gang {fit} N={N} D={D} shape {shape}")
    monkeypatch.setenv("PSO_GANG_SHAPE", shape)
    imp, st, hist = check(spec, (1, 24, 35))
    monkeypatch.delenv("PSO_GANG_SHAPE")
    monkeypatch.setenv("PSO_GANG", "0")
    imp0, st0, hist0 = check(spec, (60,))
    assert imp == imp0 and np.array_equal(hist, hist0)


@pytest.mark.parametrize("fit,N,D,tol", [("sphere", 300, 1, 1e-6), ("sphere", 5000, 2, 1e-8), ("rastrigin", 2000, 3, 1e-3),
                                         ("ackley", 700, 5, 1e-3), ("sphere", 3000, 12, 1e-3), ("sphere", 513, 20, 1.0)])
def test_gang_blocks_and_stop_rule(fit, N, D, tol):
    """Long enough for the blocks of iterations to grow (the gbest settles),
    with a stop rule that is met inside one."""
    spec = wl.SwarmSpec(fit, N, D, 900, seed=5 * N + D, shift_amplitude=1.0)
    announce(f"gang stop rule {fit} N={N} D={D}")
    check(spec, (7, 893), tol=tol)
    check(spec, (400, 500))


@pytest.mark.parametrize("name,kw", [
    ("no cognitive term", dict(c1=0.0)), ("tiny c1", dict(c1=1e-33)), ("smallest c2", dict(c2=1e-38)),
    ("lower bound 0", dict(box=(0.0, 7.0), vmax=0.7)), ("upper bound -0", dict(box=(-7.0, -0.0), vmax=0.7)),
    ("lower bound -0", dict(box=(-0.0, 7.0), vmax=3.0)), ("wide box", dict(box=(-3e6, 3e6), vmax=6e5)),
    ("infinite velocities", dict(w=3e38, vmax=1e4))])
@pytest.mark.parametrize("fit", ["rastrigin", "sphere"])
def test_gang_parameter_limits(monkeypatch, fit, name, kw):
    spec = wl.SwarmSpec(fit, 700, 6, 40, seed=11, **kw)
    announce(f"gang limits {fit}: {name}")
    imp, st, hist = check(spec, (15, 25))
    monkeypatch.setenv("PSO_GANG", "0")
    imp0, st0, hist0 = check(spec, (40,))
    assert imp == imp0
    # a state the caller set: zeros of both signs and a pbest outside the box
    with gpu_swarm(spec) as g:
        st0 = g.state()
        st0["x"][::3] = -0.0
        st0["v"][::3] = -0.0
        st0["p"][::5] = np.float32(1e3)
        out = []
        for env in ("0", None):
            monkeypatch.setenv("PSO_GANG", env) if env else monkeypatch.delenv("PSO_GANG")
            g.set_state(st0)
            g.run(20)
            out.append(g.state())
    for k in ("x", "v", "p", "pf"):
        assert np.array_equal(out[0][k].view(np.uint32), out[1][k].view(np.uint32)), k


def state64_equal(g, o):
    st = g.state()
    assert st["t"] == o["iters"] and st["gbest_idx"] == o["gbest_idx"]
    for k in ("x", "v", "p", "pf"):
        assert np.array_equal(st[k].view(np.uint64), o[k].view(np.uint64)), k


def swarm64(sp):
    return pso.Swarm64(sp.fitness, sp.N, sp.D, sp.box, sp.w, sp.c1, sp.c2, sp.vmax, sp.seed, shift=sp.shift)


@pytest.mark.parametrize("fit,N,D,shape", [
    ("cubic", 1, 1, "1,64"), ("sphere", 700, 1, "1,256"), ("rosenbrock", 1000, 2, "2,256"), ("cubic", 90, 4, "4,128"),
    ("sphere", 3000, 3, "4,1024"), ("rosenbrock", 700, 8, "8,512"), ("cubic", 300, 15, "16,256"),
    ("rosenbrock", 600, 31, "32,512"), ("sphere", 130, 5, "2,64"), ("cubic", 200, 6, "4,64"),
    ("rosenbrock", 300, 33, "8,64"), ("sphere", 129, 47, "16,128"), ("rosenbrock", 150, 70, "32,128"),
    ("rosenbrock", 50, 21, "2,32"), ("cubic", 41, 30, "4,44"), ("rosenbrock", 63, 101, "8,16")])
def test_gang64_shapes_equal_oracle(monkeypatch, fit, N, D, shape):
    T = 60
    spec = wl.SwarmSpec(fit, N, D, T, seed=N * 5 + D, shift_amplitude=1.5)
    announce(f"gang f64 {fit} N={N} D={D} shape {shape}")
    monkeypatch.setenv("PSO64_GANG_SHAPE", shape)
    o = oracle_swarm(spec, 8).run_f64(T)
    with swarm64(spec) as g:
        g.step(3)  # pending pbest positions of the grid steps before it
        g.run(20)
        r = g.run(T - 23)
        assert r["gbest_fit"] == o["gbest_fit"] and r["gbest_iter"] == o["giter"]
        state64_equal(g, o)


@pytest.mark.parametrize("fit,N,D,tol", [("sphere", 5000, 1, 1e-12), ("sphere", 700, 2, 1e-20),
                                         ("rosenbrock", 900, 3, 1e-4), ("sphere", 2000, 10, 1e-6), ("cubic", 200, 3, 0.0)])
def test_gang64_blocks_and_stop_rule(fit, N, D, tol):
    spec = wl.SwarmSpec(fit, N, D, 900, seed=5 * N + D, shift_amplitude=1.0)
    announce(f"gang f64 stop rule {fit} N={N} D={D}")
    for t in (tol, 0.0):
        o = oracle_swarm(spec, 8).run_f64(900, tol=t, f_star=0.0)
        with swarm64(spec) as g:
            r1 = g.run(7, tol=t)
            r2 = g.run(893, tol=t)
            assert r1["iters"] + r2["iters"] == o["iters"] and r2["gbest_iter"] == o["giter"]
            state64_equal(g, o)


@pytest.mark.parametrize("fit", ["rastrigin", "ackley"])
@pytest.mark.parametrize("N,D,shape", [(300, 1, "1,64"), (300, 2, "2,128"), (200, 7, "2,16"), (200, 30, "4,64"),
                                       (200, 30, "16,64"), (100, 61, "8,16"), (200, 64, "32,64")])
def test_gang64_transcendental_equals_grid_steps(monkeypatch, fit, N, D, shape):
    """Rastrigin and Ackley call the device's cos and exp: the gang's bits are
    the grid steps'."""
    spec = wl.SwarmSpec(fit, N, D, 50, seed=N + D, shift_amplitude=1.5)
    announce(f"gang f64 {fit} N={N} D={D} shape {shape}")
    out = []
    for env in (shape, None):
        if env:
            monkeypatch.setenv("PSO64_GANG_SHAPE", env)
        else:
            monkeypatch.setenv("PSO64_PATH", "grid")
        with swarm64(spec) as g:
            g.run(50)
            out.append(g.state())
    for k in ("x", "v", "p", "pf"):
        assert np.array_equal(out[0][k].view(np.uint64), out[1][k].view(np.uint64)), k
    assert out[0]["gbest_idx"] == out[1]["gbest_idx"]


@pytest.mark.parametrize("box", [(0.0, 7.0), (-7.0, -0.0), (-0.0, 7.0)])
def test_gang64_zero_bounds(box):
    spec = wl.SwarmSpec("sphere", 700, 6, 60, seed=3, box=box)
    announce(f"gang f64 bounds {box}")
    o = oracle_swarm(spec, 8).run_f64(60)
    with swarm64(spec) as g:
        g.run(60)
        state64_equal(g, o)


def test_gangs_that_exclude_each_other(monkeypatch):
    """Several swarms whose gangs each want most compute units, run from
    several threads at once: whichever parts are not resident together in time
    leave the state alone and the step launches run instead."""
    specs = [wl.SwarmSpec("rosenbrock", 65536, 40, 30, seed=s) for s in range(3)]
    monkeypatch.setenv("PSO_GANG", "0")
    want = []
    for sp in specs:
        with gpu_swarm(sp) as g:
            g.run(sp.T)
            want.append(g.state())
    monkeypatch.delenv("PSO_GANG")
    swarms = [gpu_swarm(sp) for sp in specs]
    try:
        for _ in range(2):
            for g in swarms:
                g.reset()
            errs = []

            def go(g, sp):
                try:
                    g.run(sp.T // 2)
                    g.run(sp.T - sp.T // 2)
                except Exception as e:  # noqa: BLE001 - reported below
                    errs.append(e)

            ts = [threading.Thread(target=go, args=a) for a in zip(swarms, specs)]
            [t.start() for t in ts]
            [t.join() for t in ts]
            assert not errs
            for g, w in zip(swarms, want):
                st = g.state()
                assert st["t"] == w["t"] and st["gkey"] == w["gkey"]
                for k in ("x", "v", "p", "pf"):
                    assert np.array_equal(st[k].view(np.uint32), w[k].view(np.uint32)), k
    finally:
        for g in swarms:
            g.close()


def test_gang_on_the_callers_stream():
    """pso_create_in: the caller's memory and stream, next to other work of
    that stream."""
    import torch

    spec = wl.SwarmSpec("ackley", 3000, 30, 50, seed=4, shift_amplitude=2.0)
    st = torch.cuda.Stream()
    ws = torch.zeros(pso.pso_workspace_bytes(spec.N, spec.D) + 256, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    off = (-ws.data_ptr()) % 256
    with torch.cuda.stream(st):
        a = torch.randn(512, 512, device="cuda")
        with pso.Swarm(spec.fitness, spec.N, spec.D, spec.box, spec.w, spec.c1, spec.c2, spec.vmax, spec.seed,
                       shift=spec.shift, workspace=ws[off:], stream=st) as g:
            b = a @ a
            g.run(spec.T)
            s = g.state()
            assert torch.equal(b, a @ a)
    assert_state_equal(s, oracle_swarm(spec, 8).run_f32(spec.T), spec.N, spec.D)


@pytest.mark.parametrize("fit,N,D,shape", [("rastrigin", 200, 30, "8,64"), ("sphere", 4001, 12, "2,32"), ("rosenbrock", 150, 19, "4,152"),
                                           ("ackley", 300, 66, "64,256")])
def test_stopped_gang_keeps_the_pending_marks(monkeypatch, fit, N, D, shape):
    """Steps leave pbest positions pending in x; a run whose stop rule already
    holds runs no iteration and leaves the flushed state, in both precisions."""
    spec = wl.SwarmSpec(fit, N, D, 4, seed=N + D, shift_amplitude=1.5)
    announce(f"stopped gang {fit} N={N} D={D} shape {shape}")
    c, p = shape.split(",")
    monkeypatch.setenv("PSO_GANG_SHAPE", shape)
    monkeypatch.setenv("PSO64_GANG_SHAPE", shape if int(c) <= 32 else "16,64")
    for make, bits in ((gpu_swarm, np.uint32), (swarm64, np.uint64)):
        out = []
        for run in (False, True):
            with make(spec) as g:
                g.step(4)
                if run:
                    assert g.run(10, tol=1e30)["iters"] == 0
                out.append(g.state())
        assert out[0]["t"] == out[1]["t"] == 4
        for k in ("x", "v", "p", "pf"):
            assert np.array_equal(out[0][k].view(bits), out[1][k].view(bits)), k


@pytest.mark.parametrize("fit,N,D", [("rosenbrock", 343, 10), ("sphere", 512, 12), ("rosenbrock", 511, 9)])
def test_one_part_of_eight_dimensions_a_lane(fit, N, D):
    """Sizes that take one part of wide chunks while they settle, and several
    parts once the run ends later."""
    spec = wl.SwarmSpec(fit, N, D, 900, seed=N + D, shift_amplitude=1.0)
    announce(f"one part {fit} N={N} D={D}")
    check(spec, (60, 840))
