"""Batched jobs on tiles (several sweeps per launch), by walks along z and whole
in one tile: bit-exact against the oracle run of each job alone, for calls that
leave every remainder of a tile launch's four sweeps, shapes with ragged last
tiles and columns, arenas with room for one lattice copy only, and a limit on
the work list."""
import numpy as np
import pytest

import paper_1209_0296_amd as S
from helpers import run_oracle

pytestmark = pytest.mark.gpu

JOBS = [
    S.Params(L=32, T=2.2, seed=1), S.Params(L=128, two_s=2, T=1.7, seed=2), S.Params(L=136, T=2.4, h=0.1, seed=3),
    S.Params(L=520, two_s=2, T=1.6, seed=4), S.Params(L=1000, T=2.3, seed=5),
    S.Params(model=S.NORTH_EAST, L=200, c=0.2, seed=6), S.Params(model=S.NORTH_EAST, L=1000, c=0.6, seed=7),
    S.Params(model=S.NE_COUPLED, L=400, c=0.5, T=3.0, seed=8), S.Params(model=S.NE_COUPLED, L=64, c=0.5, T=3.0, seed=9),
    S.Params(dim=3, L=16, two_s=2, T=3.0, seed=10), S.Params(dim=3, L=24, T=4.4, seed=11),
    S.Params(dim=3, L=32, two_s=2, T=3.1, seed=12), S.Params(dim=3, L=72, T=4.6, h=0.05, seed=13),
    S.Params(dim=3, L=104, two_s=2, T=3.2, seed=14), S.Params(dim=3, L=128, T=4.5, seed=15),
]


@pytest.mark.parametrize("flags", [0, S.BATCH_NO_GRAPH, S.BATCH_NO_RESIDENT])
def test_tiled_jobs_match_each_job_alone(flags):
    b = S.Batch(arena_bytes=128 << 20, max_jobs=24, record_capacity=32, flags=flags)
    budget = [13 + i % 6 for i in range(len(JOBS))]
    ids = [b.add(p, sweeps=n) for p, n in zip(JOBS, budget)]
    assert all(i is not None for i in ids)
    recs = {i: [] for i in ids}
    for n in (1, 2, 3, 4, 5, 30):
        b.sweep(n)
        for i, r in b.drain().items():
            recs[i].append(r)
    for i, p, n in zip(ids, JOBS, budget):
        print(f"case batch tiles flags={flags} job {i} model={p.model} dim={p.dim} L={p.L}", flush=True)
        assert b.status(i)[:2] == (n, 0)
        o_s, o_r = run_oracle(p, n)
        np.testing.assert_array_equal(np.vstack(recs[i]), o_r)
        np.testing.assert_array_equal(b.spins(i), o_s)
    b.close()


@pytest.mark.parametrize("p", [S.Params(dim=3, L=72, T=4.6, seed=3), S.Params(L=936, two_s=2, T=1.6, seed=4)])
def test_an_arena_of_exactly_the_reported_bytes_admits_the_job(p):
    """sl_batch_job_bytes is what a job needs at least: with no room for a second
    lattice copy it runs on one."""
    cfg = S.batch_config(max_jobs=2, record_capacity=16)
    b = S.Batch(S.batch_base_bytes(cfg) + S.batch_job_bytes(p, cfg), max_jobs=2, record_capacity=16)
    i = b.add(p, sweeps=7)
    assert i is not None
    b.sweep(3)
    b.sweep(4)
    o_s, o_r = run_oracle(p, 7)
    np.testing.assert_array_equal(S.records_to_array(b.measure(i)), o_r)
    np.testing.assert_array_equal(b.spins(i), o_s)
    b.close()


def test_a_work_list_limit_keeps_the_classes_that_fit_it():
    p = S.Params(L=1024, T=2.3, seed=6)
    b = S.Batch(32 << 20, max_jobs=2, record_capacity=16, max_workgroups=64)
    i = b.add(p, sweeps=5)
    b.sweep(5)
    o_s, o_r = run_oracle(p, 5)
    np.testing.assert_array_equal(S.records_to_array(b.measure(i)), o_r)
    np.testing.assert_array_equal(b.spins(i), o_s)
    b.close()


@pytest.mark.parametrize("jobs", [
    [S.Params(dim=3, L=72, T=4.6, seed=3), S.Params(dim=3, L=40, T=4.4, seed=5), S.Params(dim=3, L=72, two_s=2, T=3.1, seed=7)],
    [S.Params(L=936, two_s=2, T=1.6, seed=4), S.Params(dim=3, L=64, T=4.5, seed=6), S.Params(L=104, T=2.2, seed=8)]])
def test_an_arena_of_the_sum_of_the_reported_bytes_admits_every_job(jobs):
    """Second lattice copies give way to new jobs, also while one holds the state."""
    cfg = S.batch_config(max_jobs=len(jobs), record_capacity=16)
    room = S.batch_base_bytes(cfg) + sum(S.batch_job_bytes(p, cfg) for p in jobs)
    b = S.Batch(room, max_jobs=len(jobs), record_capacity=16)
    ids, recs = [], {}
    for p in jobs:
        i = b.add(p, sweeps=3 * len(jobs))
        assert i is not None
        ids.append(i)
        recs[i] = []
        b.sweep(3)
        for k in ids:
            recs[k].append(S.records_to_array(b.measure(k)))
    for n in (5, 1, 3):
        b.sweep(n)
        for k in ids:
            recs[k].append(S.records_to_array(b.measure(k)))
    for i, p in zip(ids, jobs):
        o_s, o_r = run_oracle(p, 3 * len(jobs))
        np.testing.assert_array_equal(np.vstack(recs[i]), o_r)
        np.testing.assert_array_equal(b.spins(i), o_s)
    b.close()


def test_tiles_do_not_overflow_the_default_work_list():
    """3000 jobs of 2D L = 1760 are 1.09 million tiles, more than the default work list
    of 2^20 holds; in the row class, which the same arena always had room for, 330
    thousand strips.  Every job is the same lattice, so one oracle run checks all; the
    last 120 are added when the others' state lies in the tiles' second copy."""
    p, n, late = S.Params(L=1760, T=2.3, seed=9), 3000, 120
    cfg = S.batch_config(max_jobs=n, record_capacity=8)
    second = 2 * ((p.nsites // 2 + 255) // 256 * 256)
    b = S.Batch(S.batch_base_bytes(cfg) + n * (S.batch_job_bytes(p, cfg) + second), max_jobs=n, record_capacity=8)
    for _ in range(n - late):
        assert b.add(p, sweeps=5) is not None
    b.sweep(2)
    for _ in range(late):
        assert b.add(p, sweeps=5) is not None
    b.sweep(3)
    b.sweep(2)
    got = b.drain()
    o_s, o_r = run_oracle(p, 5)
    assert len(got) == n
    for r in got.values():
        np.testing.assert_array_equal(r, o_r)
    for i in (0, n // 2, n - 1):
        np.testing.assert_array_equal(b.spins(i), o_s)
    b.close()


@pytest.mark.parametrize("p", [S.Params(dim=3, L=72, T=4.6, seed=3), S.Params(L=936, two_s=2, T=1.6, seed=4)])
def test_a_second_copy_is_lent_again_when_room_comes_free(p):
    """A job whose second copy a new job took writes one again once that job is gone:
    a lattice copy of the free arena space, marked before, is then overwritten."""
    cfg = S.batch_config(max_jobs=2, record_capacity=16)
    base, one = S.batch_base_bytes(cfg), S.batch_job_bytes(p, cfg)
    b = S.Batch(base + 2 * one, max_jobs=2, record_capacity=16)
    i = b.add(p, sweeps=14)
    b.sweep(3)
    k = b.add(p, sweeps=14)
    b.sweep(2)
    b.arena.cpu()  # nothing runs from here on
    assert k is not None
    b.remove(k)
    free = b.arena[base + one:]
    free.fill_(0x55)
    b.sweep(1)
    assert int((free != 0x55).sum()) >= 0.9 * p.nsites
    b.sweep(3)
    k = b.add(p, sweeps=14)  # taken once more, while it may hold the state
    b.sweep(5)
    for j, n in ((i, 14), (k, 5)):
        o_s, o_r = run_oracle(p, n)
        np.testing.assert_array_equal(S.records_to_array(b.measure(j)), o_r)
        np.testing.assert_array_equal(b.spins(j), o_s)
    b.close()


@pytest.mark.parametrize("p", [S.Params(dim=3, L=288, two_s=2, T=3.1, seed=3), S.Params(dim=3, L=288, T=4.5, seed=4)])
def test_large_3d_jobs_on_row_groups_or_walks(p):
    """Spin-1 rows of 63 of a wave's lanes keep the row groups, spin-1/2 ones walk."""
    b = S.Batch(256 << 20, max_jobs=2, record_capacity=8)
    i = b.add(p, sweeps=2)
    b.sweep(2)
    o_s, o_r = run_oracle(p, 2)
    np.testing.assert_array_equal(S.records_to_array(b.measure(i)), o_r)
    np.testing.assert_array_equal(b.spins(i), o_s)
    b.close()


@pytest.mark.parametrize("flags", [0, S.BATCH_NO_FUSED, S.BATCH_NO_RESIDENT])
def test_spin_one_jobs_with_zero_thresholds(flags):
    """Tables with thresholds of zero keep the row classes: fused rows, walks (without
    the fused class) and 3D row groups, of every width, beside ordinary jobs."""
    jobs = [S.Params(dim=dim, L=L, two_s=2, T=0.2, h=0.05, seed=L) for dim, L in
            ((2, 64), (2, 520), (2, 528), (2, 544), (2, 1000), (3, 32), (3, 56), (3, 72), (3, 64))]
    jobs += [S.Params(L=264, two_s=2, T=1.7, seed=1), S.Params(dim=3, L=40, two_s=2, T=3.1, seed=2)]
    assert 0 in S.threshold_table(jobs[0]) and 0 in S.threshold_table(jobs[5])
    b = S.Batch(64 << 20, max_jobs=len(jobs), record_capacity=16, flags=flags)
    ids = [b.add(p, sweeps=7) for p in jobs]
    for n in (3, 4):
        b.sweep(n)
    got = b.drain()
    for i, p in zip(ids, jobs):
        print(f"case zero thresholds flags={flags} dim={p.dim} L={p.L} T={p.T}", flush=True)
        o_s, o_r = run_oracle(p, 7)
        np.testing.assert_array_equal(got[i], o_r)
        np.testing.assert_array_equal(b.spins(i), o_s)
    b.close()


@pytest.mark.parametrize("flags", [0, S.BATCH_NO_GRAPH])
def test_short_calls_of_large_batches_run_on_rows(flags):
    """Calls of few sweeps over enough sites leave the tiles for the row classes (fused
    rows and, of one copy, walks), in place in whichever copy holds the state, and
    longer calls take the tiles again."""
    jobs = [S.Params(L=2048, T=2.3, seed=i) for i in range(8)] + [S.Params(L=1536, T=2.1, h=0.1, seed=20)]
    jobs += [S.Params(L=1024, T=2.3, seed=30 + i) for i in range(28)]
    jobs += [S.Params(L=1024, two_s=2, T=1.7, seed=60), S.Params(L=1056, two_s=2, T=1.6, seed=61),
             S.Params(model=S.NORTH_EAST, L=1024, c=0.3, seed=62), S.Params(model=S.NORTH_EAST, L=1088, c=0.2, seed=63),
             S.Params(model=S.NE_COUPLED, L=1024, c=0.5, T=3.0, seed=64), S.Params(L=72, T=2.2, seed=65),
             S.Params(L=1000, T=2.2, seed=66), S.Params(dim=3, L=64, T=4.5, seed=67)]
    assert sum(p.nsites for p in jobs) > 2 ** 26
    b = S.Batch(1 << 30, max_jobs=len(jobs), record_capacity=32, flags=flags)
    ids = [b.add(p, sweeps=17 if i % 5 else 11) for i, p in enumerate(jobs)]
    recs = {i: [] for i in ids}
    for n in (1, 3, 1, 2, 4, 5, 7):
        b.sweep(n)
        for i, r in b.drain().items():
            recs[i].append(r)
    for k, (i, p) in enumerate(zip(ids, jobs)):
        print(f"case short calls flags={flags} job {k} model={p.model} L={p.L}", flush=True)
        n = 17 if k % 5 else 11
        o_s, o_r = run_oracle(p, n)
        np.testing.assert_array_equal(np.vstack(recs[i]), o_r)
        np.testing.assert_array_equal(b.spins(i), o_s)
    b.close()
