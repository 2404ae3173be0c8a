"""The list build over bricks of cells where its cut can go wrong: windows staged in several
pieces (more atoms around a brick than the stage holds), bricks with more centers than threads
and with a few (several lanes per center, several blocks per brick), bricks that span a whole
axis, empty bricks, and replicas of different sizes and fillings in one batch.  Neighbour sets
against the oracle, bit-exact; the relative cells of the FP32-mixed entries through the forces."""
import numpy as np
import pytest

import oracle as O
from paper_1507_07068_amd import inputs as I
from paper_1507_07068_amd import md
from tests.test_gpu_parity import MIXED_TOL, check_lists, force_errors

pytestmark = pytest.mark.gpu


def uneven_gas(n, lengths, seed, periodic=(True, True, True)):
    """Half of the atoms in the lowest sixth of the box along z, the rest anywhere."""
    s = I.random_gas(n, 0.0, seed, periodic=periodic, lengths=lengths)
    s.x[::2, 2] = np.abs(s.x[::2, 2]) % (lengths[2] / 6.0)
    return s


def gas(kind, seed):
    if kind == "sparse":     # a few atoms per brick, many bricks empty
        return I.random_gas(300, 0.0, seed, periodic=(True, True, False), lengths=(60.0, 22.0, 47.0)), 32
    if kind == "uneven":     # brick and window sizes far from the average they are cut for
        return uneven_gas(6000, (27.0, 26.0, 40.0), seed), 1024
    if kind == "uneven_open":
        return uneven_gas(5000, (60.0, 18.0, 14.0), seed, periodic=(False, True, True)), 1024
    s = I.random_gas(4000, 0.0, seed, lengths=(27.0, 35.0, 28.0))   # one-cell bricks, windows in pieces
    s.potential = "paper"
    return s, 1024


@pytest.mark.parametrize("kind", ["sparse", "uneven", "uneven_open", "long_range"])
@pytest.mark.parametrize("tpa,list_tgt", [(1, 0), (4, 64)])
def test_brick_lists(kind, tpa, list_tgt):
    s, cap = gas(kind, 31)
    print(f"[case] {kind} n={s.n} cap={cap} tpa={tpa} list_tgt={list_tgt}", flush=True)
    sim = md.Simulation(s, cap=cap, tpa=tpa, list_tgt=list_tgt)
    sim.md_build_neighbors(force=True)
    st = sim.md_check()
    assert st["overflow"] == 0 and st["sync_timeout"] == 0, st
    assert check_lists(sim, s, cap=cap) > 0


def test_brick_lists_of_a_batch():
    reps = [gas("sparse", 41)[0], gas("uneven", 42)[0], I.bulk(5, seed=43), gas("uneven_open", 44)[0]]
    print(f"[case] batch {[s.n for s in reps]}", flush=True)
    b = md.Simulation(reps, cap=1024, tpa=2)
    b.md_build_neighbors(force=True)
    assert b.md_check()["overflow"] == 0
    for r, s in enumerate(reps):
        cnt, idx = O.neighbors(s, s.r_list, x=O.wrap(s), cap=1024)
        assert b.neighbor_sets(r) == O.neighbor_sets(cnt, idx), r


@pytest.mark.parametrize("list_tgt", [0, 32])
def test_brick_relative_cells(list_tgt):
    """FP32-mixed forces over the shadow (separations from the entries' relative cells) of a bulk
    with five cells per edge, whose bricks span whole axes."""
    s = I.bulk(8, seed=45, noise=0.05)
    print(f"[case] relative cells n={s.n} list_tgt={list_tgt}", flush=True)
    sim = md.Simulation(s, precision="mixed", tpa=2, list_tgt=list_tgt)
    sim.initial_forces()
    ref = O.evaluate(s, O.wrap(s))
    rel, mx = force_errors(sim.state()[0]["f"], ref["f"])
    print(f"  force rel-RMS {rel:.3e} max/RMS {mx:.3e}", flush=True)
    assert rel <= MIXED_TOL
