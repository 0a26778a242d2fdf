"""Runs beside each other: a run that takes the whole device lets others in
between its launches, and one that finds the device taken goes on and comes
back to the chip; all compute what they compute alone."""
import threading
import time

import numpy as np
import pytest

from paper_2205_01313_amd import workloads as wl
from tests.gpu_util import announce, gpu_swarm

pytestmark = pytest.mark.gpu


def test_small_runs_beside_a_run_on_every_compute_unit():
    """At most a few of the large run's launches (10 ms each) pass before a
    small run is done; launches of 50 ms made it wait 49 ms."""
    big_spec = wl.SwarmSpec("rastrigin", 262144, 30, 10000, seed=9)
    small_spec = wl.SwarmSpec("sphere", 1000, 2, 200, seed=1)
    announce("small runs beside a large one")
    with gpu_swarm(big_spec) as big, gpu_swarm(small_spec) as small:
        want = small.run(small_spec.T)
        alone = big.run(big_spec.T)
        big.reset()
        out, times = [], []
        th = threading.Thread(target=lambda: out.append(big.run(big_spec.T)))
        th.start()
        while th.is_alive():
            small.reset()
            t0 = time.perf_counter()
            r = small.run(small_spec.T)
            times.append(time.perf_counter() - t0)
            assert r["gbest_fit"] == want["gbest_fit"] and np.array_equal(r["gbest_pos"], want["gbest_pos"])
        th.join()
        assert out[0]["gbest_fit"] == alone["gbest_fit"] and out[0]["gbest_iter"] == alone["gbest_iter"]
        assert np.array_equal(out[0]["gbest_pos"], alone["gbest_pos"])
        n = big.run_paths()
    print(f"median {1e3 * np.median(times[:-1] or times):.2f} ms of {len(times)}, paths of the large run {n}", flush=True)
    assert np.median(times[:-1] or times) < 0.035
    # whatever it met, the large run came back to the chip
    assert n["resident"] + n["other"] == 2 * big_spec.T and n["resident"] >= big_spec.T + big_spec.T // 4


def test_runs_of_several_launches_equal_the_step_launches(monkeypatch):
    """Long enough for several launches, whose lengths depend on time: gang of
    one part and of many, held, both precisions, with the state read after."""
    import paper_2205_01313_amd as pso

    def make64(sp):
        return pso.Swarm64(sp.fitness, sp.N, sp.D, sp.box, sp.w, sp.c1, sp.c2, sp.vmax, sp.seed)

    for spec, make, off, path in (
            (wl.SwarmSpec("rastrigin", 65536, 64, 2000, seed=1), gpu_swarm, ("PSO_GANG", "0"), "resident"),
            (wl.SwarmSpec("sphere", 600, 2, 60000, seed=2), gpu_swarm, ("PSO_GANG", "0"), "resident"),
            (wl.SwarmSpec("ackley", 1 << 19, 48, 300, seed=3), gpu_swarm, ("PSO_GANG", "0"), "held"),
            (wl.SwarmSpec("cubic", 16384, 100, 1500, seed=4), make64, ("PSO64_PATH", "grid"), "resident"),
            (wl.SwarmSpec("sphere", 1 << 18, 32, 400, seed=5), make64, ("PSO64_PATH", "grid"), "held")):
        announce(f"several launches {spec.fitness} N={spec.N} D={spec.D} T={spec.T}")
        with make(spec) as g:
            r = g.run(spec.T)
            n, st = g.run_paths(), g.state()
        assert n[path] == spec.T
        monkeypatch.setenv(*off)
        with make(spec) as g:
            r0 = g.run(spec.T)
            assert g.run_paths()["other"] == spec.T
            st0 = g.state()
        monkeypatch.delenv(off[0])
        assert r["gbest_fit"] == r0["gbest_fit"] and r["gbest_iter"] == r0["gbest_iter"]
        for k in st0:
            assert np.array_equal(np.asarray(st[k]), np.asarray(st0[k])), k


def test_run_that_finds_the_device_taken_comes_back_to_the_chip():
    """Matrix products on another stream hold the compute units at first: the
    parts that are not resident together leave, other launches go on, and once
    the products are done the run is on the chip again; held and resident."""
    import torch

    import paper_2205_01313_amd as pso

    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    side = torch.cuda.Stream()
    for spec, make, path in ((wl.SwarmSpec("rastrigin", 262144, 30, 12000, seed=9), gpu_swarm, "resident"),
                             (wl.SwarmSpec("sphere", 1 << 19, 48, 2500, seed=3), gpu_swarm, "held"),
                             (wl.SwarmSpec("cubic", 16384, 100, 10000, seed=4), None, "resident")):
        announce(f"beside matrix products: {spec.fitness} N={spec.N} D={spec.D}")
        if make is None:
            g = pso.Swarm64(spec.fitness, spec.N, spec.D, spec.box, spec.w, spec.c1, spec.c2, spec.vmax, spec.seed)
        else:
            g = make(spec)
        with g:
            alone = g.run(spec.T)
            g.reset()
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                for _ in range(40):
                    b = a @ a
            r = g.run(spec.T)
            n = g.run_paths()
            torch.cuda.synchronize()
            print(f"paths {n}", flush=True)
        assert sum(n.values()) == 2 * spec.T and n[path] >= spec.T + spec.T // 4
        assert r["gbest_fit"] == alone["gbest_fit"] and r["gbest_iter"] == alone["gbest_iter"]
        assert np.array_equal(r["gbest_pos"], alone["gbest_pos"])
    assert torch.equal(b, a @ a)
