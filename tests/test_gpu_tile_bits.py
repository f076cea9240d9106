"""Tiles of bit words (large North-East lattices, J = 0, c <= 1/2): bit-exact against
the oracle at the first sizes that take them, rows that are and are not whole 16-byte
pieces, ragged last tiles, no draws at all and draws nearly everywhere, with chunks
that leave remainders of a launch's sweeps."""
import numpy as np
import pytest

import paper_1209_0296_amd as S
from helpers import run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,c,kw", [
    (1440, 0.1, {}), (1448, 0.3, {}), (1536, 0.499, {}), (2056, 0.5, {}),
    (2072, 0.02, dict(seed=2 ** 40 + 5, t0=11)), (4104, 0.2, {})])
def test_bit_tiles(L, c, kw):
    chunks = [1, 2, 13] if L < 4000 else [3]
    p = S.Params(**{**dict(model=S.NORTH_EAST, L=L, c=c, seed=L + 3, record_capacity=32), **kw})
    got_s, got_r = run_gpu(p, sum(chunks), chunks=chunks)
    ref_s, ref_r = run_oracle(p, sum(chunks))
    np.testing.assert_array_equal(got_r, ref_r)
    np.testing.assert_array_equal(got_s, ref_s)


def test_persistence_survives_the_bits():
    """Flags set before, a reset between, and a copy that continues."""
    p = S.Params(model=S.NORTH_EAST, L=1448, c=0.25, seed=9, record_capacity=32)
    a = S.Lattice(p)
    a.sweep(5)
    a.reset_persistence()
    a.sweep(3)
    one = S.records_to_array(a.measure())
    spins = a.spins()
    a.close()
    b = S.Lattice(p)
    b.set_launch(S.MODE_SIMPLE)
    b.sweep(5)
    b.reset_persistence()
    b.sweep(3)
    np.testing.assert_array_equal(one, S.records_to_array(b.measure()))
    np.testing.assert_array_equal(spins, b.spins())
    b.close()
