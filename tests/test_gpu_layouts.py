"""Lattices in and out of the natural order, and the record and overlap of a
lattice as it is: caller buffers at any byte alignment, rows of odd and even
word counts, against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
import paper_1209_0296_amd as S
import workloads as W
from helpers import oracle_params

pytestmark = pytest.mark.gpu

SHAPES = [dict(L=8), dict(L=40, two_s=2), dict(L=520), dict(dim=3, L=8, two_s=2), dict(dim=3, L=24),
          dict(model=S.NORTH_EAST, L=72, c=0.3), dict(model=S.NE_COUPLED, L=136, c=0.5, T=3.0)]


@pytest.mark.parametrize("offset", [0, 1, 4])
@pytest.mark.parametrize("kw", SHAPES)
def test_buffers_at_any_alignment(kw, offset):
    p = S.Params(seed=3, init=S.INIT_BUFFER, record_capacity=4, **kw)
    spins = W.random_lattice(p.shape, p.two_s, seed=7, model=p.model, flag_fraction=0.4)
    dev = torch.zeros(p.nsites + 16, dtype=torch.int8, device="cuda")
    dev[offset:offset + p.nsites] = torch.from_numpy(spins.reshape(-1)).cuda()
    lat = S.Lattice(p, init_spins=dev[offset:offset + p.nsites])
    ref = O.initial_record(oracle_params(p), spins)
    if p.model == S.ISING:
        ref[4] = -1
    np.testing.assert_array_equal(S.records_to_array(lat.measure())[0], ref)
    out = torch.full((p.nsites + 16,), 55, dtype=torch.int8, device="cuda")
    status = S.lib().sl_copy_spins(lat._h, out.data_ptr() + offset, ctypes.c_size_t(p.nsites))
    assert status == 0
    host = out.cpu().numpy()
    np.testing.assert_array_equal(host[offset:offset + p.nsites], spins.reshape(-1))
    assert (host[:offset] == 55).all() and (host[offset + p.nsites:] == 55).all()
    other = W.random_lattice(p.shape, p.two_s, seed=8, model=p.model).astype(np.int64).reshape(-1)
    dev[offset:offset + p.nsites] = torch.from_numpy(other.astype(np.int8)).cuda()
    v = spins.reshape(-1).astype(np.int64)
    if p.model != S.ISING:
        v, other = 2 * (v & 1) - 1, 2 * (other & 1) - 1
    assert lat.overlap(dev[offset:offset + p.nsites]) == int((v * other).sum())
    lat.close()
