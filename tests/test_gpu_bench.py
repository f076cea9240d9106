"""What bench.py reports of a schedule that runs several sweeps per launch."""
import pytest
import torch

import bench
import paper_1209_0296_amd as S
from workloads import CONFIGS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,launches", [("ne2d_L4096", 2), ("ising2d_L64", 1), ("ising2d_L8192", 24),
                                           ("ising3d_L256_s12", 48)])
def test_launches_and_bytes_are_those_of_the_kernels_that_run(name, launches):
    """24 sweeps: North-East 4096 in two launches of tiles, 2D L = 64 whole in one, the
    others by the schedule that get_launch names.  A launch of tiles reads and writes
    the lattice once, so no schedule moves more than the memory can."""
    steps = 24
    r = bench.time_workload(S, torch, name, CONFIGS[name], steps, 12)
    assert r["launch"]["launches_per_sweep"] * steps == pytest.approx(launches)
    assert r["launch"]["sweeps_per_launch"] == pytest.approx(steps / launches)
    lattice = 2 * r["nsites"] * (1 if launches != 48 else 0.5)
    assert r["roofline"]["algo_bytes_per_launch"] == lattice
    assert 0 < r["roofline"]["frac"] < 1
