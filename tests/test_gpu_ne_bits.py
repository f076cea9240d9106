"""GPU parity of the sub-lattice kernels where the lattice changes its form: one
sweep per call (colour arrays to bit rows and back), several, every sub-lattice
side, one sub-lattice, a partial workgroup, the fewest steps per launch, and
thresholds that are never met."""
import numpy as np
import pytest

import paper_1209_0296_amd as S
from helpers import run_gpu, run_oracle

pytestmark = pytest.mark.gpu

CASES = [(side, lam, L) for side, lam, L in [
    (8, 2, 8), (8, 8, 40), (16, 4, 16), (16, 16, 80), (32, 2, 96), (32, 64, 64),
    (64, 2, 128), (64, 4, 64), (64, 32, 192)]]


@pytest.mark.parametrize("model", [S.NE_SUBLATTICE, S.NE_SUBLATTICE_BALANCED], ids=["random", "balanced"])
@pytest.mark.parametrize("side,lam,L", CASES)
def test_calls_of_one_and_more_sweeps(model, side, lam, L):
    p = S.Params(model=model, L=L, ne_side=side, ne_lambda=lam, c=0.35, seed=5 * L + side + lam)
    g_s, g_r = run_gpu(p, 5, chunks=[1, 3, 1])
    o_s, o_r = run_oracle(p, 5)
    np.testing.assert_array_equal(g_r, o_r)
    np.testing.assert_array_equal(g_s, o_s)


@pytest.mark.parametrize("c", [1e-12, 1.0 - 1e-12], ids=["no_up", "no_down"])
@pytest.mark.parametrize("model", [S.NE_SUBLATTICE, S.NE_SUBLATTICE_BALANCED], ids=["random", "balanced"])
def test_a_threshold_of_zero(model, c):
    p = S.Params(model=model, L=64, ne_side=16, ne_lambda=8, c=c, seed=23)
    g_s, g_r = run_gpu(p, 4, chunks=[1, 3])
    o_s, o_r = run_oracle(p, 4)
    np.testing.assert_array_equal(g_r, o_r)
    np.testing.assert_array_equal(g_s, o_s)


@pytest.mark.parametrize("B,lam,balanced", [
    (B, lam, balanced) for B in (16, 32, 64) for lam in (32, 64, 128) for balanced in (False, True)
    if (8 if balanced else 2) * lam <= B * B])
def test_columns_put_together_by_ballots(B, lam, balanced):
    """16, 32 and 64 lanes a sub-lattice, more and fewer than its rows, one sub-lattice
    to a wavefront and several: the east columns of the colour arrays and of the rows
    that pass between a call's launches."""
    for L in (B, 2 * B, 5 * B):
        p = S.Params(model=S.NE_SUBLATTICE_BALANCED if balanced else S.NE_SUBLATTICE, L=L, c=0.45, seed=B + lam + L,
                     ne_side=B, ne_lambda=lam, record_capacity=16)
        got_s, got_r = run_gpu(p, 5, chunks=[1, 3, 1])
        ref_s, ref_r = run_oracle(p, 5)
        np.testing.assert_array_equal(got_r, ref_r)
        np.testing.assert_array_equal(got_s, ref_s)
