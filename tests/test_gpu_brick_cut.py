"""List build on a grid of a very long axis (120,000 list cells), on the device: pairs of atoms strewn
along it, neighbour sets against the oracle."""
import numpy as np
import pytest

from paper_1507_07068_amd import inputs as I
from paper_1507_07068_amd import md
from tests.test_gpu_parity import check_lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_long_axis(axis):
    lengths = np.full(3, 13.0)
    lengths[axis] = 504_100.0
    s = I.random_gas(3000, 0.0, 47 + axis, lengths=lengths)
    s.x[1::2] = s.x[::2] + np.random.default_rng(axis).uniform(-2.5, 2.5, s.x[::2].shape)
    print(f"[case] long axis {axis} n={s.n}", flush=True)
    sim = md.Simulation(s, tpa=2)
    sim.md_build_neighbors(force=True)
    st = sim.md_check()
    assert st["overflow"] == 0 and st["sync_timeout"] == 0, st
    assert check_lists(sim, s) > s.n // 2
