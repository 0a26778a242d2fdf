"""Which path ran: the shapes and sizes that the tests of the resident gang,
the held runs and the register-held batches force or expect take that path (all
paths compute the same bits, so those tests alone cannot tell)."""
import pytest

import paper_2205_01313_amd as pso
from paper_2205_01313_amd import workloads as wl
from tests import test_gpu_gang, test_gpu_hold, test_gpu_resident
from tests.gpu_util import announce, gpu_swarm

pytestmark = pytest.mark.gpu


def cases_of(test, names):
    """The values a test function is parametrised with."""
    for mark in test.pytestmark:
        if mark.name == "parametrize" and mark.args[0] == names:
            return mark.args[1]
    raise AssertionError(names)


def paths_of(g, T):
    g.run(T)
    n = g.run_paths()
    assert sum(n.values()) == T
    return n


def test_forced_gang_shapes_run_resident(monkeypatch):
    announce("forced gang shapes")
    for fit, N, D, shape in cases_of(test_gpu_gang.test_gang_shapes_equal_oracle, "fit,N,D,shape"):
        monkeypatch.setenv("PSO_GANG_SHAPE", shape)
        with gpu_swarm(wl.SwarmSpec(fit, N, D, 20, seed=N)) as g:
            assert paths_of(g, 20)["resident"] == 20, (fit, N, D, shape)


def test_forced_binary64_gang_shapes_run_resident(monkeypatch):
    announce("forced binary64 gang shapes")
    forced = [(f, *c) for c in cases_of(test_gpu_gang.test_gang64_transcendental_equals_grid_steps, "N,D,shape")
              for f in ("rastrigin", "ackley")]
    forced += cases_of(test_gpu_gang.test_gang64_shapes_equal_oracle, "fit,N,D,shape")
    for fit, N, D, shape in forced:
        monkeypatch.setenv("PSO64_GANG_SHAPE", shape)
        with test_gpu_gang.swarm64(wl.SwarmSpec(fit, N, D, 20, seed=N)) as g:
            assert paths_of(g, 20)["resident"] == 20, (fit, N, D, shape)


def test_chosen_gangs_run_resident():
    """The sizes of the tests that leave the choice to the rule."""
    announce("chosen gangs")
    for name, make in (("test_gang_blocks_and_stop_rule", gpu_swarm), ("test_gang64_blocks_and_stop_rule", test_gpu_gang.swarm64)):
        for fit, N, D, _ in cases_of(getattr(test_gpu_gang, name), "fit,N,D,tol"):
            with make(wl.SwarmSpec(fit, N, D, 100, seed=N)) as g:
                assert paths_of(g, 100)["resident"] == 100, (fit, N, D)


def test_held_runs_are_held(monkeypatch):
    announce("held runs")
    with gpu_swarm(wl.SwarmSpec("rastrigin", 1 << 19, 48, 40, seed=5)) as g: # chosen by the rule
        assert paths_of(g, 20)["held"] == 20
    monkeypatch.setenv("PSO_HOLD", "1")
    monkeypatch.setenv("PSO_GANG_SHAPE", "0,0")
    for k, (N, D) in enumerate(test_gpu_hold.SIZES):
        with gpu_swarm(wl.SwarmSpec(wl.FITNESS_NAMES[k % 5], N, D, 5, seed=k)) as g:
            assert paths_of(g, 5)["held"] == 5, (N, D)
    monkeypatch.setenv("PSO64_GANG_SHAPE", "0,0")
    for fit, N, D in cases_of(test_gpu_hold.test_held_runs_in_binary64, "fit,N,D"):
        sp = wl.SwarmSpec(fit, N, D, 5, seed=N)
        with pso.Swarm64(fit, N, D, sp.box, sp.w, sp.c1, sp.c2, sp.vmax, 7) as g:
            assert paths_of(g, 5)["held"] == 5, (fit, N, D)


def test_switched_off_paths_do_not_run(monkeypatch):
    announce("paths switched off")
    monkeypatch.setenv("PSO_GANG", "0")
    with gpu_swarm(wl.SwarmSpec("sphere", 3000, 12, 30, seed=1)) as g:
        assert paths_of(g, 30) == dict(resident=0, held=0, other=30)


@pytest.mark.parametrize("name", list(test_gpu_resident.EDGES))
def test_batches_of_the_edges_are_held_in_registers(name):
    announce(f"register-held batch: {name}")
    with pso.Batch(test_gpu_resident.specs_of(name)) as b:
        assert b.in_registers
        b.set_shape(256, 0, 1 << 17)
        assert not b.in_registers


# T of the runs that stay off the resident gang, and the first T on it
@pytest.mark.parametrize("fit,N,D,off,on", [
    ("sphere", 262144, 8, (1, 2, 4), 6), ("sphere", 131072, 2, (1, 4), 8), ("cubic", 262144, 1, (7,), 10), ("ackley", 131072, 30, (1,), 2),
    ("rastrigin", 262144, 30, (1, 4), 5), ("cubic", 36000, 43, (2, 3), 4), ("sphere", 262144, 30, (1, 3), 4), ("rosenbrock", 4000, 30, (1,), 2), ("cubic", 16384, 2, (), 1),
    ("sphere", 641, 2, (60, 200, 400), 500), ("rosenbrock", 1300, 2, (50, 300), 500), ("sphere", 640, 2, (), 200),
    ("cubic", 31, 25, (4, 100), None), ("rastrigin", 16, 17, (300,), None), ("cubic", 8, 250, (100,), None), ("sphere", 32, 25, (), 1),
    ("sphere", 17, 24, (), 1), ("ackley", 600, 2, (50, 199), 200), ("ackley", 900, 1, (50, 100), 200), ("rastrigin", 641, 2, (), 60), ("sphere", 800, 3, (), 60)])
def test_runs_too_short_for_the_gang(fit, N, D, off, on):
    """Runs that the step launches or the one-workgroup run finish sooner (the
    state's way on and off the chip, or a meeting in most iterations)."""
    announce(f"short runs {fit} N={N} D={D}")
    with gpu_swarm(wl.SwarmSpec(fit, N, D, 1, seed=N + D)) as g:
        for T in off:
            g.reset()
            g.run(T)
        assert g.run_paths() == dict(resident=0, held=0, other=sum(off))
        if on is None:
            return
        g.reset()
        g.run(on)
        assert g.run_paths() == dict(resident=on, held=0, other=sum(off))


@pytest.mark.parametrize("N,D,registers", [(256, 2, True), (257, 2, False), (1025, 2, True), (64, 3, False), (300, 3, False), (640, 8, False),
                                           (641, 8, True), (512, 16, False), (513, 16, True), (257, 17, True), (300, 5, False)])
def test_one_swarm_batches_in_registers(N, D, registers):
    """A swarm that has the device to itself, on both sides of the lines
    between the 1024-lane workgroup and parts that meet."""
    announce(f"batch of one swarm N={N} D={D}")
    with pso.Batch([wl.SwarmSpec("rastrigin", N, D, 10, seed=N)]) as b:
        assert b.in_registers == registers


def test_run_that_goes_on_is_not_short():
    """What the short runs' rule is for is over when a swarm has settled: a
    short run 500 iterations after Step 1 stays on the chip, after a reset not."""
    announce("short run of a settled swarm")
    with gpu_swarm(wl.SwarmSpec("sphere", 1000, 2, 1, seed=3)) as g:
        g.run(600)
        g.run(100)
        assert g.run_paths() == dict(resident=700, held=0, other=0)
        g.reset()
        g.run(100)
        assert g.run_paths() == dict(resident=700, held=0, other=100)
        g.step(400)
        g.run(100)
        assert g.run_paths() == dict(resident=800, held=0, other=100)
