"""Performance cases: what a user of the library has it do, each through its
public entry points, at sizes from one iteration of a small swarm to the
largest single swarm, ragged sizes among them, in binary32 and binary64.

A case is a dict of plain values.  Its "kind" says which entry points run:
  step    Swarm.reset, Swarm.step, Swarm.best: one binary32 iteration
  run     Swarm.reset, Swarm.run, Swarm.history: a whole binary32 solve and its
          convergence curve; with "checkpoint" Swarm.state too
  run64   Swarm64.reset, Swarm64.run: a whole binary64 solve
  batch   Batch.launch, Batch.results: uneven swarms in one launch
  serve   Server.submit, Server.poll: a burst of solve requests
"""
from __future__ import annotations

import numpy as np
import torch

import paper_2205_01313_amd as pso
from paper_2205_01313_amd import workloads as wl

# Shift amplitude of a drawn or listed problem: within its box, so that the
# optimum is not at the centre of the search range.
SHIFT = {"sphere": 20.0, "rastrigin": 2.0, "rosenbrock": 2.0, "ackley": 10.0, "cubic": 0.0}


def listed():
    return [
        # the smallest call: one iteration of the small Sphere swarm and its
        # gbest, as a caller that steers a swarm from its own loop does
        dict(name="step_sphere_d2_n1024", kind="step", fitness="sphere", N=1024, D=2, T=1, tol=0.0, f_star=0.0),
        # the small Sphere workload: a solve of milliseconds
        dict(name="run_sphere_d2_n1024", kind="run", fitness="sphere", N=1024, D=2, T=1000, tol=0.0, f_star=0.0),
        # synchronous latency at D = 1 (the paper's Cubic problem, binary32)
        dict(name="run_cubic_d1_n16384", kind="run", fitness="cubic", N=16384, D=1, T=2000, tol=0.0, f_star=0.0),
        # a ragged swarm of few dimensions with a precision target (the stop
        # rule is tested every iteration; this target is out of reach), its
        # state saved at the end
        dict(name="run_rastrigin_d11_n5001", kind="run", fitness="rastrigin", N=5001, D=11, T=500, tol=1e-4,
             f_star=-1.0, checkpoint=True),
        # the usual test-function size: 30 dimensions, a few thousand particles
        dict(name="run_ackley_d30_n2000", kind="run", fitness="ackley", N=2000, D=30, T=500, tol=0.0, f_star=0.0,
             checkpoint=True),
        # the deep workload: many dimensions, a state of 100 MB
        dict(name="run_rosenbrock_d128_n65536", kind="run", fitness="rosenbrock", N=65536, D=128, T=200, tol=0.0,
             f_star=0.0),
        # the large Rastrigin workload, whole: the largest state
        dict(name="run_rastrigin_d32_n1048576", kind="run", fitness="rastrigin", N=1 << 20, D=32, T=200, tol=0.0,
             f_star=0.0),
        # the paper's own precision and problem, one dimension
        dict(name="run64_cubic_d1_n16384", kind="run64", fitness="cubic", N=16384, D=1, T=2000, tol=0.0, f_star=0.0),
        # the paper's 120-dimensional shape
        dict(name="run64_cubic_d120_n8192", kind="run64", fitness="cubic", N=8192, D=120, T=200, tol=0.0,
             f_star=0.0),
        # a large binary64 swarm (double cos)
        dict(name="run64_rastrigin_d32_n262144", kind="run64", fitness="rastrigin", N=1 << 18, D=32, T=50, tol=0.0,
             f_star=0.0),
        # many independent uneven swarms in one launch
        dict(name="batch_256", kind="batch", count=256, T=500, mix=0),
        # a burst of solve requests to the server, each with its stop rule
        dict(name="serve_200", kind="serve", count=200, T=1000, mix=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))


# Particle-dimension updates of a drawn solve at most (the large Rastrigin
# workload has 6.7e9), and its iterations.
MAX_UPDATES = 4e9


def draw(rng):
    kind = rng.choice(["step", "run", "run", "run", "run", "run64", "run64", "batch", "serve"])
    if kind == "batch":
        return dict(kind=kind, count=_log_int(rng, 16, 256), T=rng.randint(100, 500),
                    mix=rng.randint(1, 1 << 20))
    if kind == "serve":
        return dict(kind=kind, count=_log_int(rng, 20, 200), T=rng.randint(200, 1000),
                    mix=rng.randint(1, 1 << 20))
    fitness = rng.choice(["sphere", "rastrigin", "rosenbrock", "ackley", "cubic"])
    D = _log_int(rng, 2 if fitness == "rosenbrock" else 1, 128)
    N = _log_int(rng, 32, (1 << 18) if kind == "run64" else (1 << 20))
    per = float(N * D)
    most = (MAX_UPDATES / 8 if kind == "run64" else MAX_UPDATES) / per
    T = 1 if kind == "step" else int(max(10, min(2000 if D <= 2 else 500, most) * rng.uniform(0.5, 1.0)))
    stop = kind != "step" and rng.random() < 0.25
    case = dict(kind=kind, fitness=fitness, N=N, D=D, T=T, tol=1e-4 if stop else 0.0, f_star=-1.0 if stop else 0.0)
    if kind == "run" and N * D <= 100000 and rng.random() < 0.25:
        case["checkpoint"] = True
    return case


def _problem(case, seed):
    """Parameters of a single swarm: fitness, box, w, c1, c2, vmax, shift."""
    f = case["fitness"]
    box = wl.BOX[f]
    # the paper's experiments state w = 1, c1 = c2 = 2 for Cubic; the others
    # take the usual constriction coefficients
    w, c1, c2 = (1.0, 2.0, 2.0) if f == "cubic" else (wl.W, wl.C1, wl.C2)
    shift = wl.shift_vector(seed, case["D"], SHIFT[f]) if SHIFT[f] > 0 else None
    return box, w, c1, c2, wl.vmax_of(box), shift


def _specs(case, seed):
    """The swarms of a batch or burst: sizes and functions of its mix, shift
    vectors and Philox seeds of the seed."""
    if case["kind"] == "batch":
        specs = wl.batch_specs(case["count"], seed=case["mix"], T=case["T"])
    else:
        specs = wl.serving_specs(case["count"], seed=case["mix"], max_iter=case["T"])
    for k, sp in enumerate(specs):
        sp.seed = seed * 100003 + k
        sp.shift = wl.shift_vector(sp.seed, sp.D, 5.0)
    return specs


def prepare(case, seed):
    seed = int(seed)
    kind = case["kind"]
    if kind == "batch":
        return dict(case=case, batch=pso.Batch(_specs(case, seed)))
    if kind == "serve":
        return dict(case=case, specs=_specs(case, seed), server=pso.Server(1 << 30))
    box, w, c1, c2, vmax, shift = _problem(case, seed)
    cls = pso.Swarm64 if kind == "run64" else pso.Swarm
    return dict(case=case, swarm=cls(case["fitness"], case["N"], case["D"], box, w, c1, c2, vmax, seed, shift=shift))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        state["batch"].launch()
        return _columns(state["batch"].results())
    if kind == "serve":
        srv = state["server"]
        pending = [srv.submit(sp) for sp in state["specs"]]
        done = {}
        order = list(pending)
        while pending:
            still = []
            for t in pending:
                r = srv.poll(t)
                if r is None:
                    still.append(t)
                else:
                    done[t] = r
            pending = still
        return _columns([done[t] for t in order])
    g = state["swarm"]
    g.reset()
    if kind == "step":
        g.step()
        return g.best()
    r = g.run(case["T"], tol=case["tol"], f_star=case["f_star"])
    if kind == "run":
        r["history"] = g.history(0, r["iters"] + 1)
        if case.get("checkpoint"):
            r["state"] = g.state()
            r["state"]["gkey"] = np.uint64(r["state"]["gkey"])
    return r


def _columns(results):
    """The results of many swarms, one array per field."""
    return dict(gbest_fit=np.array([r["gbest_fit"] for r in results]),
                gbest_iter=np.array([r["gbest_iter"] for r in results]),
                iters=np.array([r["iters"] for r in results]),
                gbest_pos=np.concatenate([r["gbest_pos"] for r in results]))


# Arithmetic of one particle-dimension update: Philox4x32-10 yields the draws
# of two dimensions with 20 32x32-bit products and 40 exclusive-ors; Eq. 1 and
# its clamp 11, Eq. 2 and its clamp 3, the two uniforms 4; then the fitness.
FIT_FLOPS = {"sphere": 3, "rastrigin": 24, "rosenbrock": 8, "ackley": 24, "cubic": 9}
ON_CHIP = 160e6  # bytes of registers and LDS: a larger state passes through memory every iteration


def _solve_work(fitness, N, D, T, word):
    state = 3.0 * word * N * D
    per_iter = 5.0 * word * N * D if state > ON_CHIP else 0.0
    return 2.0 * state + T * per_iter, float(N) * D * T * (30 + 18 + FIT_FLOPS[fitness])


def work(case):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        both = [_solve_work(sp.fitness, sp.N, sp.D, sp.T, 4) for sp in _specs(case, 0)]
        return dict(bytes=float(sum(b for b, _ in both)), flops=float(sum(f for _, f in both)))
    b, f = _solve_work(case["fitness"], case["N"], case["D"], case["T"], 8 if kind == "run64" else 4)
    return dict(bytes=b, flops=f)


# ---------------------------------------------------------------------------
# The method in plain torch, in 64 bits.
# ---------------------------------------------------------------------------
M32 = 0xFFFFFFFF


def _philox(k0, k1, c0, c1, t, tag):
    """Philox4x32-10 over int64 tensors that hold 32-bit words."""
    c0, c1 = torch.broadcast_tensors(c0, c1)
    c2, c3 = torch.full_like(c0, t), torch.full_like(c0, tag)
    for _ in range(10):
        m0, m1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # wraps modulo 2^64: the low 64 bits
        c0, c1, c2, c3 = ((m1 >> 32) & M32) ^ c1 ^ k0, m1 & M32, ((m0 >> 32) & M32) ^ c3 ^ k1, m0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _draws(seed, N, D, t, tag, dev):
    """Two uniforms in [0, 1) per (dimension, particle), 24 bits each."""
    pairs = (D + 1) // 2
    c0 = torch.arange(pairs, device=dev, dtype=torch.int64)[:, None]
    c1 = torch.arange(N, device=dev, dtype=torch.int64)[None, :]
    a, b, c, d = _philox(seed & M32, (seed >> 32) & M32, c0, c1, t, tag)
    u1 = torch.stack((a, c), 1).reshape(2 * pairs, N)[:D]
    u2 = torch.stack((b, d), 1).reshape(2 * pairs, N)[:D]
    return (u1 >> 8).double() * 2.0**-24, (u2 >> 8).double() * 2.0**-24


def _cospi(y):
    n = torch.round(y)
    c = torch.cos(np.pi * (y - n))
    return torch.where(torch.remainder(n, 2.0) != 0.0, -c, c)


def _fitness(f, z):
    D = z.shape[0]
    acc, aux = torch.zeros_like(z[0]), torch.zeros_like(z[0])
    if f == "sphere":
        for d in range(D):
            acc = acc + z[d] * z[d]
        return acc
    if f == "rastrigin":
        term = z * z - 10.0 * _cospi(2.0 * z)
        for d in range(D):
            acc = acc + term[d]
        return 10.0 * D + acc
    if f == "rosenbrock":
        for d in range(1, D):
            a, b = z[d] - z[d - 1] * z[d - 1], 1.0 - z[d - 1]
            acc = acc + (100.0 * a * a + b * b)
        return acc
    if f == "ackley":
        s, c = z * z, _cospi(2.0 * z)
        for d in range(D):
            acc, aux = acc + s[d], aux + c[d]
        return 20.0 - 20.0 * torch.exp(-0.2 * torch.sqrt(acc / D)) + np.e - torch.exp(aux / D)
    term = z * z * z - 0.8 * z * z - 1000.0 * z + 8000.0
    for d in range(D):
        acc = acc + term[d]
    return -acc


def exact(case, seed):
    """Binary64 solves, and one iteration of binary32 ones, in 64 bits.  None
    for longer binary32 solves, batches and requests: the strict pbest test
    turns on the last binary32 bit, so within some iterations a 64-bit solve
    is a different trajectory and no value of that one."""
    kind = case["kind"]
    if kind not in ("step", "run64"):
        return None
    seed = int(seed)
    N, D, T = case["N"], case["D"], case["T"]
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    seconds = T * ((60 + 4 * D) * 12e-6 + N * D * 150 * 1e-11) if dev.type == "cuda" else N * D * T * 150 * 1e-9
    if seconds > 15.0:
        return None
    box, w, c1, c2, vmax, shift = _problem(case, seed)
    lo, hi, w, c1, c2, vmax = (float(np.float32(v)) for v in (*box, w, c1, c2, vmax))
    s = torch.zeros(D, dtype=torch.float64) if shift is None else torch.from_numpy(shift.astype(np.float64))
    s = s.to(dev)[:, None]
    u0, u1 = _draws(seed, N, D, 0, 1, dev)
    x = (lo + (hi - lo) * u0).clamp(lo, hi)
    v = (-vmax + 2.0 * vmax * u1).clamp(-vmax, vmax)
    p, pf = x.clone(), _fitness(case["fitness"], x - s)
    best, gi = torch.min(pf, 0)
    best, gpos, giter = float(best), p[:, int(gi)].clone(), 0
    for t in range(1, T + 1):
        r1, r2 = _draws(seed, N, D, t, 0, dev)
        v = (w * v + c1 * r1 * (p - x) + c2 * r2 * (gpos[:, None] - x)).clamp(-vmax, vmax)
        x = (x + v).clamp(lo, hi)
        f = _fitness(case["fitness"], x - s)
        better = f < pf
        pf = torch.where(better, f, pf)
        p = torch.where(better[None, :], x, p)
        m = float(torch.min(pf))
        if m < best:
            gi = int(torch.nonzero(pf == m)[0])
            best, gpos, giter = m, p[:, gi].clone(), t
    if kind == "step":
        return dict(gbest_fit=best, gbest_pos=gpos.cpu().numpy(), gbest_iter=None, t=None)
    return dict(gbest_fit=best, gbest_pos=gpos.cpu().numpy(), gbest_iter=None, iters=None)
