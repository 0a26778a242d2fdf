"""The batched kernel whose parts hold their particles in registers, at the
edges of its split (one part and many, one to four lanes per particle, odd D,
a part of one particle), bit for bit against the streamed shape and the
oracle; resumed launches through the server; and what it refuses."""
import numpy as np
import pytest

import paper_2205_01313_amd as pso
from paper_2205_01313_amd import workloads as wl
from tests.gpu_util import announce, oracle_swarm

pytestmark = pytest.mark.gpu

EDGES = {
    # D: chunks of 2 to 16 dimensions, the last one full or not
    "D": [(N, D) for N in (63, 257, 700) for D in (1, 2, 3, 15, 16, 17, 31, 33, 47, 49, 63, 64)],
    # N: lanes per particle by N, one part or many, the last of one particle
    "N": [(N, D) for N in (1, 2, 64, 65, 128, 129, 193, 256, 513) for D in (1, 7, 12, 16, 18, 32, 40)],
    "many parts": [(20001, 2), (4097, 17), (6001, 48), (8193, 64), (16385, 16), (30000, 1)],
}


def specs_of(name, T=40):
    out = []
    for k, (N, D) in enumerate(EDGES[name]):
        for fit in wl.FITNESS_NAMES[:5] if name != "many parts" else (wl.FITNESS_NAMES[k % 5],):
            if fit == "rosenbrock" and D < 2:
                continue
            sp = wl.SwarmSpec(fit, N, D, T - k % 7 if k % 11 else 0, seed=1000 * N + D, shift_amplitude=1.5)
            if k % 3 == 0:
                sp.tol, sp.f_star = (1e-1, 0.0) if fit != "cubic" else (1e3, -8e5 * D)
            out.append(sp)
    return out


def same(res, ref, specs):
    for sp, r, q in zip(specs, res, ref):
        assert r["gbest_fit"] == q["gbest_fit"] and r["gbest_iter"] == q["gbest_iter"], sp
        assert r["iters"] == q["iters"] and np.array_equal(r["gbest_pos"], q["gbest_pos"]), sp


@pytest.mark.parametrize("name", list(EDGES))
def test_register_parts_equal_streamed_and_oracle(name):
    specs = specs_of(name)
    announce(f"register-held parts: {name}, {len(specs)} swarms")
    with pso.Batch(specs) as b:
        full = b.shape
        outs = []
        for grid in (0, 248 if name == "many parts" else 3):  # full grid; the work queue runs long
            b.set_shape(full["lanes"], grid, 0, stage_kib=full["stage_kib"])
            for _ in range(2):
                b.launch()
                outs.append(b.results())
        b.set_shape(256, 0, 1 << 17)
        b.launch()
        ref = b.results()
    for res in outs:
        same(res, ref, specs)
    for k in range(0, len(specs), 5 if name != "many parts" else 2):
        sp = specs[k]
        o = oracle_swarm(sp, 8).run_f32(sp.T, tol=getattr(sp, "tol", 0.0), f_star=getattr(sp, "f_star", 0.0))
        assert outs[0][k]["gbest_fit"] == o["gbest_fit"] and outs[0][k]["gbest_iter"] == o["giter"], sp
        assert outs[0][k]["iters"] == o["iters"] and np.array_equal(outs[0][k]["gbest_pos"], o["gpos"]), sp


@pytest.mark.parametrize("name", list(EDGES))
def test_register_parts_resume_in_the_server(name):
    """The server runs a request in slices, so its state leaves the registers
    and comes back: chunks of a few iterations give what one launch gives."""
    specs = specs_of(name, T=23)
    announce(f"register-held parts, resumed: {name}")
    ref = pso.pso_batch_run(specs)
    with pso.Server(1 << 29, chunk_updates=1 << 16) as srv:
        tickets = [srv.submit(sp) for sp in specs]
        res = []
        for t in tickets:
            r = None
            while r is None:
                r = srv.poll(t)
            res.append(r)
    same(res, ref, specs)


@pytest.mark.parametrize("change", [dict(c1=1e-33), dict(c2=-1e-35), dict(box=(-1.0, -0.0)), dict(shift_amplitude=3e6)])
def test_parameters_the_short_forms_do_not_cover(change):
    """One such swarm sends its whole batch to the LDS-staged kernel; the
    results stay those of the streamed shape and the oracle."""
    specs = [wl.SwarmSpec("rastrigin", 70, 7, 30, seed=70, **{"shift_amplitude": 1.0, **change}),
             wl.SwarmSpec("ackley", 300, 7, 30, seed=300, shift_amplitude=1.0)]
    announce(f"batch with {change}")
    with pso.Batch(specs) as b:
        b.launch()
        res = b.results()
        b.set_shape(256, 0, 1 << 17)
        b.launch()
        same(res, b.results(), specs)
    for sp, r in zip(specs, res):
        o = oracle_swarm(sp, 8).run_f32(sp.T)
        assert r["gbest_fit"] == o["gbest_fit"] and np.array_equal(r["gbest_pos"], o["gpos"]), sp
