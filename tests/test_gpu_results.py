"""Results reach the host whatever else the thread has done."""
import ctypes

import numpy as np
import pytest

import paper_2205_01313_amd as pso
from paper_2205_01313_amd import workloads as wl
from tests.gpu_util import announce, gpu_swarm, oracle_swarm

pytestmark = pytest.mark.gpu


def test_results_after_an_unrelated_error():
    """A failed call elsewhere (an allocation larger than any device) leaves the
    thread an error to read; reading a swarm's results is not refused for it."""
    spec = wl.SwarmSpec("rastrigin", 300, 5, 20, seed=3, shift_amplitude=1.0)
    announce("results after an unrelated error")
    hip = pso.lib()
    o = oracle_swarm(spec, 8).run_f32(20)
    with gpu_swarm(spec) as g:
        g.step(20)
        p = ctypes.c_void_p()
        assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 50)) != 0
        try:
            g.sync()
            best = g.best()
            counters, history = g.counters(), g.history(0, 21)
        finally:
            hip.hipGetLastError()
    assert best["gbest_fit"] == o["gbest_fit"] and best["gbest_iter"] == o["giter"]
    assert np.array_equal(best["gbest_pos"], o["gpos"]) and np.array_equal(history, o["hist"])
    assert counters["pbest_improvements"] > 0
