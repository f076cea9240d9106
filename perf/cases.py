"""Work that a user of this package has it do, as measurable cases.

A pass of a `run` case advances a lattice that the program keeps on the GPU by
a chunk of sweeps, drains the per-sweep records and takes a copy of the
lattice: the loop of every simulation script, whose chunk is what lies between
two looks at the records.  A pass of a `restart` case is a whole short
simulation: a lattice is created from spins in a device buffer (a checkpoint,
or a start made elsewhere), swept, measured, copied and closed.  A pass of a
`serve` case hands a closed batch of independent jobs to the job server and
collects every job's records.

Ranges: 2D Ising lattices from L = 32 to 8192 and 3D ones from 16 to 256, spin
1/2 and 1, with and without a field, temperatures of 0.8 to 1.2 of the critical
one; North-East lattices by checkerboard, with the Ising coupling and by random
sub-lattices up to L = 4096.  L is any multiple of 8, as the package takes it.

Every output is a whole number (spins and counts), so there is nothing that
64-bit arithmetic could give more exactly: exact() has no values, and outputs
are compared for equality.
"""
import math

import numpy as np
import torch

import paper_1209_0296_amd as S
from paper_1209_0296_amd.serve import Request, Server

ISING, NORTH_EAST, NE_SUB, NE_BALANCED, NE_COUPLED = 0, 1, 2, 3, 4
# critical temperatures, used only to place the temperatures: {(dim, 2 spin)}
TC = {(2, 1): 2.0 / math.log(1.0 + math.sqrt(2.0)), (2, 2): 1.6935, (3, 1): 4.5115, (3, 2): 3.19}
MOST_ATTEMPTS = 8192 * 8192 * 100  # of one pass: the largest listed case


def _ising(dim, L, two_s, T, sweeps, h=0.0, start="random", kind="run"):
    return dict(kind=kind, model=ISING, dim=dim, L=L, two_s=two_s, J=1.0, h=h, T=T, c=0.5, start=start,
                side=32, lam=16, sweeps=sweeps)


def _ne(model, L, c, sweeps, J=1.0, h=0.0, T=3.0, side=32, lam=16):
    return dict(kind="run", model=model, dim=2, L=L, two_s=1, J=J, h=h, T=T, c=c, start="random",
                side=side, lam=lam, sweeps=sweeps)


def _serve(jobs, lo, hi, chunk, mix):
    return dict(kind="serve", jobs=jobs, sweeps_lo=lo, sweeps_hi=hi, chunk=chunk, mix=mix)


def listed():
    return [
        # the smallest run: 64 x 64 from a cold start, E and M of each of 1000 sweeps
        dict(_ising(2, 64, 1, 2.269, 1000, start="cold"), name="ising2d_L64_cold"),
        # the size the paper times its 2D code at, 512 x 512
        dict(_ising(2, 512, 1, 2.269, 200), name="ising2d_L512"),
        # a size that is no power of two (131 words a colour row), spin 1 in a field
        dict(_ising(2, 1048, 2, 1.6, 100, h=0.1), name="ising2d_L1048_s1_field"),
        # the headline lattice, 8192 x 8192 at T = 2.269
        dict(_ising(2, 8192, 1, 2.269, 100), name="ising2d_L8192"),
        # a small 3D lattice, where a sweep is shorter than its launches
        dict(_ising(3, 64, 1, 4.5115, 200), name="ising3d_L64"),
        # the 256^3 lattices, spin 1/2 and spin 1
        dict(_ising(3, 256, 1, 4.5115, 50), name="ising3d_L256_s12"),
        dict(_ising(3, 256, 2, 3.19, 50), name="ising3d_L256_s1"),
        # North-East by checkerboard, 4096 x 4096 at c = 0.1, with persistence
        dict(_ne(NORTH_EAST, 4096, 0.1, 100), name="ne2d_L4096"),
        # the same by the paper's random sub-lattices (B = 32, lambda = 16)
        dict(_ne(NE_SUB, 4096, 0.1, 20), name="ne2d_sub_L4096"),
        # the North-East constraint on the Ising energy, at an odd size (125 words a row)
        dict(_ne(NE_COUPLED, 1000, 0.5, 100), name="ne2d_coupled_L1000"),
        # a short run restarted from a saved lattice
        dict(_ising(2, 2048, 2, 1.6935, 10, kind="restart"), name="restart_L2048_s1"),
        # the served stream's mix as a closed batch; a tenth of its sweeps a job, so that a
        # pass stays short
        dict(_serve(256, 100, 1000, 64, mix=5), name="serve_256_jobs"),
    ]


def _log_size(rng, lo, hi, unit=8):
    """Log-uniform multiple of `unit` in [lo, hi]."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, unit * round(v / unit))))


def _sweeps(rng, nsites, scale=1.0):
    """A chunk of 10 to 1000 sweeps that stays within the largest listed pass."""
    most = max(10, min(1000, int(scale * MOST_ATTEMPTS / nsites / 2)))
    return int(round(math.exp(rng.uniform(math.log(10), math.log(most)))))


def draw(rng):
    kind = rng.choice(["2d", "2d", "2d", "3d", "3d", "ne", "ne", "ne_sub", "restart", "serve"])
    if kind == "serve":
        return _serve(rng.randint(16, 192), 100, rng.randint(200, 900), rng.choice([32, 64, 128]),
                      mix=rng.randrange(1 << 30))
    if kind in ("2d", "3d", "restart"):
        dim = rng.choice([2, 3]) if kind == "restart" else int(kind[0])
        L = _log_size(rng, *((32, 8192) if dim == 2 and kind != "restart" else (64, 4096) if dim == 2 else (16, 256)))
        two_s = rng.choice([1, 2])
        T = round(rng.uniform(0.8, 1.2) * TC[(dim, two_s)], 4)
        h = rng.choice([0.0, 0.0, 0.0, round(rng.uniform(-0.5, 0.5), 3)])
        n = rng.randint(2, 30) if kind == "restart" else _sweeps(rng, L ** dim)
        start = "random" if kind == "restart" else rng.choice(["random", "random", "cold"])
        return _ising(dim, L, two_s, T, n, h=h, start=start, kind="restart" if kind == "restart" else "run")
    if kind == "ne":
        L = _log_size(rng, 64, 4096)
        c = round(rng.uniform(0.05, 0.3), 3)
        n = _sweeps(rng, L * L, 0.25)
        if rng.random() < 0.3:
            return _ne(NE_COUPLED, L, 0.5, n, J=rng.choice([1.0, -1.0]), h=round(rng.uniform(0.0, 0.3), 2),
                       T=round(rng.uniform(2.0, 4.0), 3))
        return _ne(NORTH_EAST, L, c, n)
    side = rng.choice([16, 32, 32, 64])
    L = _log_size(rng, 4 * side, 4096, side)
    return _ne(rng.choice([NE_SUB, NE_SUB, NE_BALANCED]), L, round(rng.uniform(0.05, 0.42), 3),
               min(200, _sweeps(rng, L * L, 0.02)), side=side, lam=rng.choice([8, 16, 16, 32]))


def _params(case, seed):
    init = {"cold": S.INIT_COLD, "random": S.INIT_RANDOM, "buffer": S.INIT_BUFFER}
    start = "buffer" if case["kind"] == "restart" else case["start"]
    return S.Params(model=case["model"], dim=case["dim"], L=case["L"], two_s=case["two_s"], J=case["J"],
                    h=case["h"], T=case["T"], c=case["c"], seed=seed + 1, init=init[start],
                    record_capacity=case["sweeps"] + 2, ne_side=case["side"], ne_lambda=case["lam"])


def _jobs(case, seed):
    """Jobs of the served stream's mix: 2D L log-uniform in [32, 1024] or 3D L in
    [16, 128], spin 1/2 or 1, T uniform in [0.8, 1.2] T_c, a seed per job.  The mix
    is the case's; the seed makes the jobs' own random numbers."""
    rng = np.random.default_rng(case["mix"])
    out = []
    for i in range(case["jobs"]):
        dim = 2 if rng.random() < 0.5 else 3
        lo, hi = (32, 1024) if dim == 2 else (16, 128)
        L = float(np.exp(rng.uniform(np.log(lo), np.log(hi))))
        L = int(min(hi, max(lo, 8 * round(L / 8))))
        two_s = 1 if rng.random() < 0.5 else 2
        p = S.Params(dim=dim, L=L, two_s=two_s, T=float(rng.uniform(0.8, 1.2) * TC[(dim, two_s)]),
                     seed=100000 * (seed + 1) + i)
        out.append(Request(i, 0.0, p, int(rng.integers(case["sweeps_lo"], case["sweeps_hi"] + 1))))
    return out


def prepare(case, seed):
    if case["kind"] == "serve":
        server = Server(1 << 30, max_jobs=max(64, case["jobs"]), chunk=case["chunk"])
        return dict(case=case, server=server, jobs=_jobs(case, seed))
    p = _params(case, seed)
    if case["kind"] == "restart":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        shape = (case["L"],) * case["dim"]
        if case["two_s"] == 1:
            spins = 2 * torch.randint(0, 2, shape, generator=g, device="cuda", dtype=torch.int8) - 1
        else:
            spins = torch.randint(-1, 2, shape, generator=g, device="cuda", dtype=torch.int8)
        return dict(case=case, params=p, spins=spins)
    lat = S.Lattice(p)
    lat.measure()  # the record of the start
    return dict(case=case, lattice=lat)


def run(state):
    case = state["case"]
    if case["kind"] == "serve":
        outcomes, _ = state["server"].run(state["jobs"], realtime=False)
        return np.concatenate([outcomes[r.id].records for r in state["jobs"]])
    if case["kind"] == "restart":
        with S.Lattice(state["params"], init_spins=state["spins"]) as lat:
            lat.sweep(case["sweeps"])
            return dict(records=S.records_to_array(lat.measure()), spins=lat.copy_spins())
    lat = state["lattice"]
    lat.sweep(case["sweeps"])
    return dict(records=S.records_to_array(lat.measure()), spins=lat.copy_spins())


def _attempt_ops(model, two_s):
    """32-bit operations one flip attempt cannot do without: its share of the
    Philox4x32-10 calls (10 rounds of two wide products, each counted once, and
    four xors; a call gives four words, and spin 1 and the sub-lattices take
    two words an attempt), the neighbour sum, the comparison and the flip."""
    words = 2 if two_s == 2 or model in (NE_SUB, NE_BALANCED) else 1
    return words * 60.0 / 4.0 + 8.0


def work(case):
    """The lattice read once and written once, a record of 40 bytes a sweep, and
    the operations of every attempt."""
    if case["kind"] == "serve":
        jobs = _jobs(case, 0)
        sites = [r.params.nsites for r in jobs]
        return {"bytes": sum(2.0 * n + 40.0 * (r.sweeps + 1) for n, r in zip(sites, jobs)),
                "flops": sum(n * r.sweeps * _attempt_ops(ISING, r.params.two_s) for n, r in zip(sites, jobs))}
    n = float(case["L"]) ** case["dim"]
    return {"bytes": 2.0 * n + 40.0 * case["sweeps"],
            "flops": n * case["sweeps"] * _attempt_ops(case["model"], case["two_s"])}


def exact(case, seed):
    return None  # whole numbers only
