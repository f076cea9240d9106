"""Tile launches (several sweeps of LDS tiles per launch, the default schedule of
small and middle lattices): bit-exact against the oracle at the sizes where a
tile can go wrong -- the whole lattice as one tile, a dimension that a tile
spans, ragged last tiles, halos deeper than a tile, several rounds of tiles per
CU, 3D lattices up to the last tiled one -- with chunks that leave every
remainder of a launch's sweeps; walks along z, which the larger 3D lattices
take; and spin-1 tables with zero thresholds, which keep to other kernels."""
import numpy as np
import pytest

import paper_1209_0296_amd as S
from helpers import run_gpu, run_oracle

pytestmark = pytest.mark.gpu

CHUNKS = [1, 2, 3, 12, 13, 17]
KINDS = {
    "half": dict(T=2.269), "half_field": dict(T=2.0, h=-0.3, J=-1.0), "one": dict(two_s=2, T=1.7, h=0.1),
    "ne": dict(model=S.NORTH_EAST, c=0.3), "ne_half": dict(model=S.NORTH_EAST, c=0.5),
    "ne_up": dict(model=S.NORTH_EAST, c=0.6), "coupled": dict(model=S.NE_COUPLED, c=0.5, T=3.0, h=0.1),
}


def _same(sp, chunks, launch=None):
    got_s, got_r = run_gpu(sp, sum(chunks), launch=launch, chunks=chunks)
    ref_s, ref_r = run_oracle(sp, sum(chunks))
    np.testing.assert_array_equal(got_r, ref_r)
    np.testing.assert_array_equal(got_s, ref_s)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("L", [8, 40, 64, 72, 136, 264, 520])
def test_tiles_2d(L, kind):
    _same(S.Params(L=L, seed=L + 1, record_capacity=64, **KINDS[kind]), CHUNKS)


@pytest.mark.parametrize("kind", ["half", "one", "ne", "coupled"])
@pytest.mark.parametrize("L", [1048, 2056])
def test_tiles_2d_many_rounds(L, kind):
    _same(S.Params(L=L, seed=L + 1, record_capacity=16, **KINDS[kind]), [1, 3, 5])


@pytest.mark.parametrize("kw", [dict(T=4.5), dict(T=4.0, h=0.2), dict(two_s=2, T=3.1, h=-0.2)])
@pytest.mark.parametrize("L", [8, 16, 24, 40, 72, 128])
def test_tiles_3d(L, kw):
    _same(S.Params(dim=3, L=L, seed=L + 1, record_capacity=64, **kw), [1, 2, 3, 7] if L > 40 else CHUNKS)


@pytest.mark.parametrize("kw", [dict(T=4.5), dict(two_s=2, T=3.1, h=-0.2)])
@pytest.mark.parametrize("L", [136, 144, 200, 264])
def test_walks_along_z(L, kw):
    """3D lattices above the tiled ones: columns of rows walked along z, ragged
    last columns in both directions, odd and even first planes."""
    _same(S.Params(dim=3, L=L, seed=L + 1, record_capacity=64, **kw), [1, 3])


@pytest.mark.parametrize("launch", [None, (S.MODE_HALF, 4, 1), (S.MODE_FUSED, 4, 2), (S.MODE_HALF_ROWS, 4, 4)])
@pytest.mark.parametrize("dim", [2, 3])
def test_spin_one_zero_thresholds(dim, launch):
    """Tables with thresholds of zero beside ones of 2^32 and ordinary ones."""
    sp = S.Params(dim=dim, L=128 if dim == 2 else 32, two_s=2, T=0.2, h=0.05, seed=3, record_capacity=16)
    t = S.threshold_table(sp)
    assert 0 in t and 2 ** 32 in t
    if not (dim == 3 and launch is not None and launch[0] == S.MODE_FUSED):
        _same(sp, [2, 5], launch=launch)


def test_tiles_between_other_schedules():
    """The two lattice copies stay in step when schedules alternate."""
    sp = S.Params(L=256, T=2.3, seed=5, record_capacity=64)
    ref_s, ref_r = run_oracle(sp, 24)
    lat = S.Lattice(sp)
    recs = [S.records_to_array(lat.measure())]
    for mode, n in ((S.MODE_AUTO, 5), (S.MODE_FUSED, 3), (S.MODE_AUTO, 13), (S.MODE_HALF_WINDOW, 2), (S.MODE_AUTO, 1)):
        lat.set_launch(mode)
        lat.sweep(n)
        recs.append(S.records_to_array(lat.measure()))
    np.testing.assert_array_equal(np.vstack(recs), ref_r)
    np.testing.assert_array_equal(lat.spins(), ref_s)
    lat.close()


@pytest.mark.parametrize("L,kind", [(1536, "half"), (1536, "one"), (2048, "ne_up"), (2048, "coupled"), (4096, "half")])
def test_short_calls_between_tile_launches(L, kind):
    """Calls of one (or two) sweeps run on whole rows, longer ones on tiles."""
    _same(S.Params(L=L, seed=L + 5, record_capacity=16, **KINDS[kind]), [1, 3, 1, 2] if L < 4000 else [2, 3, 1])


@pytest.mark.parametrize("kw,sweeps_per_launch", [
    (dict(L=512, T=2.3), 12), (dict(dim=3, L=64, T=4.5), 3), (dict(dim=3, L=136, T=4.5), 1), (dict(L=64, T=2.3), 4096),
    (dict(model=S.NORTH_EAST, L=1536, c=0.1), None)])
def test_the_reported_schedule_set_back_changes_nothing(kw, sweeps_per_launch):
    """set_launch(*get_launch()) keeps the tiles or walks that run beside the named
    schedule; naming that schedule in plain numbers runs it."""
    lat = S.Lattice(S.Params(seed=5, record_capacity=64, **kw))
    first = lat.get_launch()
    assert first[0].sweeps_per_launch == sweeps_per_launch or sweeps_per_launch is None
    lat.set_launch(*first)
    again = lat.get_launch()
    assert again == first and again[0].sweeps_per_launch == first[0].sweeps_per_launch
    lat.set_launch(*[int(v) for v in first])
    named = lat.get_launch()
    assert named == first and not hasattr(named[0], "sweeps_per_launch")
    lat.set_launch(S.MODE_SIMPLE)
    lat.set_launch(*first)
    assert lat.get_launch()[0].sweeps_per_launch == first[0].sweeps_per_launch
    lat.sweep(9)
    got_r, got_s = S.records_to_array(lat.measure()), lat.spins()
    lat.close()
    ref_s, ref_r = run_oracle(S.Params(seed=5, **kw), 9)
    np.testing.assert_array_equal(got_r, ref_r)
    np.testing.assert_array_equal(got_s, ref_s)


@pytest.mark.parametrize("two_s,L,walks", [(1, 248, True), (1, 256, False), (1, 264, True), (1, 288, True),
                                           (2, 160, True), (2, 192, True), (2, 224, False), (2, 248, True),
                                           (2, 256, False), (2, 288, False), (2, 416, True)])
def test_3d_lattices_whose_rows_fill_their_waves_keep_the_row_groups(two_s, L, walks):
    """The choice follows the lanes of a wave that the rows fill and the waves of a
    launch, on both sides of the line; whichever runs, the lattice is the same."""
    sp = S.Params(dim=3, L=L, two_s=two_s, T=4.5 if two_s == 1 else 3.1, seed=L, record_capacity=8)
    lat = S.Lattice(sp)
    assert hasattr(lat.get_launch()[0], "sweeps_per_launch") == walks
    lat.close()
    if L in (224, 256, 288):
        _same(sp, [2])


@pytest.mark.parametrize("two_s,L", [(1, 296), (1, 344), (1, 504), (2, 248), (2, 344), (2, 496)])
def test_walks_along_z_with_two_words_a_thread(two_s, L):
    """The larger walks hold two words of a plane per thread; ragged last columns in
    both directions, up to the last size that walks."""
    sp = S.Params(dim=3, L=L, two_s=two_s, T=4.5 if two_s == 1 else 3.1, h=0.1, seed=L, record_capacity=8)
    _same(sp, [1, 1] if L < 400 else [1])


@pytest.mark.parametrize("kw", [dict(T=2.269), dict(two_s=2, T=1.7)])
def test_tiles_of_large_rows_that_fit_no_row_kernel(kw):
    """2D L = 8200: a launch of four sweeps and one of one."""
    _same(S.Params(L=8200, seed=3, record_capacity=8, **kw), [4, 1])


@pytest.mark.parametrize("kw", [dict(L=2304, T=2.3), dict(L=2560, two_s=2, T=1.7), dict(L=7168, T=2.3)])
def test_one_sweep_beyond_full_launches(kw):
    """Calls of 4 m + 1 sweeps of large lattices: one on whole rows, the rest in launches
    of four; and the widest rows below 8192, which run on rows alone."""
    _same(S.Params(seed=5, record_capacity=16, **kw), [5, 1, 9] if kw["L"] < 7000 else [3, 2])
