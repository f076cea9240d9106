"""Continuous batching: requests arriving while others run are admitted as
memory frees up, and every result equals the same lattice run alone."""
import numpy as np
import pytest

import paper_1209_0296_amd as S
from paper_1209_0296_amd.serve import Request, Server, run_one_per_launch
from helpers import run_oracle

pytestmark = pytest.mark.gpu


def _requests():
    rng = np.random.default_rng(3)
    reqs = []
    t = 0.0
    for i in range(24):
        t += rng.exponential(0.01)
        dim = 2 if i % 3 else 3
        L = int(rng.choice([32, 40, 64, 96, 128])) if dim == 2 else int(rng.choice([16, 24, 32]))
        two_s = 1 + (i % 2)
        T = (2.2 if dim == 2 else 4.3) if two_s == 1 else (1.6 if dim == 2 else 3.0)
        p = S.Params(dim=dim, L=L, two_s=two_s, T=T * float(rng.uniform(0.9, 1.1)), seed=500 + i)
        reqs.append(Request(i, t, p, int(rng.integers(20, 70))))
    return reqs


def test_served_results_equal_alone_runs():
    reqs = _requests()
    # room for only a few jobs at a time: later requests wait for retirements
    cfg = S.batch_config(max_jobs=64, record_capacity=17)
    biggest = max(S.batch_job_bytes(r.params, cfg) for r in reqs)
    arena = S.batch_base_bytes(cfg) + 3 * biggest
    srv = Server(arena, max_jobs=64, chunk=16)
    outcomes, stats = srv.run(reqs, realtime=True)
    srv.close()
    assert stats["jobs"] == len(reqs)
    base, _ = run_one_per_launch(reqs, realtime=False)
    for r in reqs:
        o_s, o_r = run_oracle(r.params, r.sweeps)
        np.testing.assert_array_equal(outcomes[r.id].records, o_r)
        np.testing.assert_array_equal(base[r.id].records, o_r)
        assert outcomes[r.id].finished >= outcomes[r.id].admitted >= 0.0
    # admission really was limited by the arena: some job waited in the queue
    waits = [outcomes[r.id].admitted - r.arrival for r in reqs]
    assert max(waits) > 0.0


def test_a_server_job_waits_for_the_second_copies_of_the_others():
    """Room for one lattice beside its second copy, but not for another lattice as
    well: the server's next job waits, where sl_batch_add admits it by its footprint."""
    p = S.Params(dim=3, L=72, T=4.6, seed=3)
    cfg = S.batch_config(max_jobs=4, record_capacity=17)
    arena = S.batch_base_bytes(cfg) + 2 * S.batch_job_bytes(p, cfg)
    srv = Server(arena, max_jobs=4, chunk=16)
    b = srv.batch
    i = b.add(p, 9)
    assert i is not None and b.add(p, 9) is None
    b.sweep(4)
    assert b.add(p, 9) is None
    b.sweep(5)
    o_s, o_r = run_oracle(p, 9)
    np.testing.assert_array_equal(S.records_to_array(b.measure(i)), o_r)
    np.testing.assert_array_equal(b.spins(i), o_s)
    b.remove(i)
    assert b.add(p, 9) is not None
    srv.close()
    plain = S.Batch(arena, max_jobs=4, record_capacity=17)
    assert plain.add(p, 9) is not None and plain.add(p, 9) is not None
    plain.close()


def test_a_server_whose_arena_holds_one_copy_of_a_job_runs_it():
    """An empty arena of exactly the footprint: the job runs in the class that needs
    no second copy."""
    p = S.Params(dim=3, L=72, T=4.6, seed=4)
    cfg = S.batch_config(max_jobs=4, record_capacity=17)
    srv = Server(S.batch_base_bytes(cfg) + S.batch_job_bytes(p, cfg), max_jobs=4, chunk=16)
    reqs = [Request(i, 0.0, p, 20) for i in range(2)]
    outcomes, _ = srv.run(reqs, realtime=False)
    srv.close()
    _, o_r = run_oracle(p, 20)
    for r in reqs:
        np.testing.assert_array_equal(outcomes[r.id].records, o_r)
