"""Runs that hold part of the state on the chip: sizes whose last lanes, parts
and dimensions are ragged, forced below the size where they are chosen, bit for
bit against the grid step (and the oracle), with continued runs, the state read
and set in between, and the stop rule."""
import numpy as np
import pytest

import paper_2205_01313_amd as pso
from paper_2205_01313_amd import workloads as wl
from tests.gpu_util import announce, assert_state_equal, gpu_swarm, oracle_swarm

pytestmark = pytest.mark.gpu

# N: one group per lane and several, lanes without one, a last group cut short;
# D: fewer pairs than are held, some streamed, some in LDS, odd
SIZES = [(70001, 3), (300001, 8), (524290, 12), (1100003, 5), (140003, 21), (131073, 26), (600001, 33), (70001, 47)]


def runs(spec, cuts, tol=0.0):
    with gpu_swarm(spec) as g:
        for n in cuts:
            r = g.run(n, tol=tol)
        st = g.state()
        hist = g.history(0, st["t"] + 1)
        return r, st, hist, g.counters()["pbest_improvements"]


@pytest.mark.parametrize("k", range(len(SIZES)))
def test_held_runs_equal_the_grid_step(monkeypatch, k):
    N, D = SIZES[k]
    spec = wl.SwarmSpec(wl.FITNESS_NAMES[k % 5], N, D, 14, seed=77 + k, shift_amplitude=1.0)
    announce(f"held run {spec.fitness} N={N} D={D}")
    monkeypatch.setenv("PSO_GANG_SHAPE", "0,0")  # no gang of this shape
    monkeypatch.setenv("PSO_HOLD", "1")          # whatever its share
    r, st, hist, imp = runs(spec, (1, 4, 9))
    monkeypatch.setenv("PSO_HOLD", "0")
    r0, st0, hist0, imp0 = runs(spec, (14,))
    assert r["gbest_fit"] == r0["gbest_fit"] and r["gbest_iter"] == r0["gbest_iter"] and imp == imp0
    assert np.array_equal(hist, hist0)
    for key in st0:
        assert np.array_equal(np.asarray(st[key]), np.asarray(st0[key])), key
    if N * D < 2_000_000:
        assert_state_equal(st, oracle_swarm(spec, 16).run_f32(14), N, D)


def test_held_run_stop_rule_and_default_choice(monkeypatch):
    """The size at which a run holds part of its state by itself, stopped by
    its rule at the iteration the grid step stops at."""
    spec = wl.SwarmSpec("rastrigin", 1 << 19, 48, 40, seed=5, shift_amplitude=0.5)
    announce("held run, stop rule")
    with gpu_swarm(spec) as g:
        f = g.run(20)["gbest_fit"]
    out = []
    for env in ("1", "0"):
        monkeypatch.setenv("PSO_HOLD", env) if env == "0" else monkeypatch.delenv("PSO_HOLD", raising=False)
        out.append(runs(spec, (40,), tol=float(f) * 1.0001))
    assert out[0][1]["t"] == out[1][1]["t"] < 40
    assert out[0][0]["gbest_fit"] == out[1][0]["gbest_fit"] and np.array_equal(out[0][2], out[1][2])


@pytest.mark.parametrize("fit,N,D", [("sphere", 60001, 3), ("rastrigin", 131072, 32), ("ackley", 262145, 27),
                                     ("rosenbrock", 70003, 40), ("cubic", 400001, 11)])
def test_held_runs_in_binary64(monkeypatch, fit, N, D):
    """Between the runs, steps of the wide and of the narrow grid step (which
    takes no pending pbest position); the reference takes wide ones only."""
    spec = wl.SwarmSpec(fit, N, D, 12, seed=N, shift_amplitude=1.0)
    announce(f"held binary64 run {fit} N={N} D={D}")
    out = []
    monkeypatch.setenv("PSO64_GANG_SHAPE", "0,0")  # no gang of this shape
    for hold in ("1", "0"):
        monkeypatch.setenv("PSO_HOLD", hold)
        with pso.Swarm64(fit, N, D, spec.box, spec.w, spec.c1, spec.c2, spec.vmax, 7,
                         shift=np.asarray(spec.shift, np.float64)) as g:
            for n in (1, 5, 6):
                r = g.run(n)
                if hold == "1":
                    monkeypatch.setenv("PSO64_WIDE", str(n % 2))
                g.step(2)
                monkeypatch.delenv("PSO64_WIDE", raising=False)
            st = g.state()
            out.append((r, st))
    (r, st), (r0, st0) = out
    assert r["gbest_fit"] == r0["gbest_fit"] and r["gbest_iter"] == r0["gbest_iter"]
    for key in st0:
        assert np.array_equal(np.asarray(st[key]), np.asarray(st0[key])), key


def test_held_runs_that_exclude_each_other():
    """Two held runs at once need every compute unit each: one waits for the
    other or takes the grid step, and both compute what they compute alone."""
    import threading

    specs = [wl.SwarmSpec("rastrigin", 1 << 19, 20, 60, seed=1, shift_amplitude=1.0),
             wl.SwarmSpec("sphere", 600001, 16, 60, seed=2, shift_amplitude=1.0)]
    announce("held runs at once")
    alone = []
    for sp in specs:
        with gpu_swarm(sp) as g:
            alone.append(g.run(sp.T))
    swarms = [gpu_swarm(sp) for sp in specs]
    out = [[], []]

    def work(k):
        for _ in range(4):
            swarms[k].reset()
            out[k].append(swarms[k].run(specs[k].T))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    for g in swarms:
        g.close()
    for k in range(2):
        assert len(out[k]) == 4
        for r in out[k]:
            assert r["gbest_fit"] == alone[k]["gbest_fit"] and r["gbest_iter"] == alone[k]["gbest_iter"]
            assert np.array_equal(r["gbest_pos"], alone[k]["gbest_pos"])


@pytest.mark.parametrize("wide,fit,N,D", [
    (False, "sphere", 2000003, 4), (False, "cubic", 4000001, 3), (False, "ackley", 70001, 511), (False, "rosenbrock", 20011, 101),
    (True, "rastrigin", 300001, 40), (True, "rosenbrock", 40001, 301), (True, "ackley", 20001, 101), (True, "cubic", 2000001, 2),
    (True, "sphere", 9001, 512)])
def test_held_runs_at_the_edges_of_what_they_accept(monkeypatch, wide, fit, N, D):
    """Four and more groups of particles a lane, up to 512 dimensions, and
    streamed rows that fit the memory-side cache or not, against the grid step."""
    spec = wl.SwarmSpec(fit, N, D, 7, seed=N + D, shift_amplitude=1.0)
    announce(f"held run {'binary64' if wide else 'binary32'} {fit} N={N} D={D}")
    monkeypatch.setenv("PSO64_GANG_SHAPE" if wide else "PSO_GANG_SHAPE", "0,0")  # no gang of this shape
    out = []
    for hold in ("1", "0"):
        monkeypatch.setenv("PSO_HOLD", hold)
        make = pso.Swarm64 if wide else pso.Swarm
        with make(fit, N, D, spec.box, spec.w, spec.c1, spec.c2, spec.vmax, 7, shift=spec.shift) as g:
            r = [g.run(n) for n in (2, 5)][-1]
            assert g.run_paths()["held"] == (7 if hold == "1" else 0)
            out.append((r, g.state()))
    (r, st), (r0, st0) = out
    assert r["gbest_fit"] == r0["gbest_fit"] and r["gbest_iter"] == r0["gbest_iter"]
    for key in st0:
        assert np.array_equal(np.asarray(st[key]), np.asarray(st0[key])), key
