"""The list build's work items: bricks that hold several blocks' worth of centers beside empty ones
(vacuum in the grid), more bricks than atoms, and batches of such replicas of which some rebuild.
Neighbour sets against the oracle, trajectories of a batch against each replica alone, bit for bit."""
import numpy as np
import pytest

import oracle as O
from paper_1507_07068_amd import inputs as I
from paper_1507_07068_amd import md
from tests.test_gpu_parity import check_lists

pytestmark = pytest.mark.gpu


def slab(nx, ny, nz, height, seed, temperature=300.0):
    """A film in a periodic box of `height` times its own: bricks of 6^3 cells, most of them empty and
    the others with over a thousand centers."""
    s = I.film(nx, ny, nz, 0.0, 0.0, seed, noise=0.05, temperature=temperature)
    s.periodic = np.array([True, True, True])
    s.box_len = s.box_len.copy()
    s.box_len[2] = nz * I.A_CR * height
    return s


def dimers(n, box, seed):
    s = I.random_gas(n, box, seed)
    u = np.random.default_rng(seed).normal(size=(n // 2, 3))
    s.x[1::2] = s.x[::2] + 2.5 * u / np.linalg.norm(u, axis=1)[:, None]
    return s


@pytest.mark.parametrize("tpa,precision", [(1, "fp64"), (4, "mixed")])
@pytest.mark.parametrize("kind", ["slab", "open", "dilute", "one_tile", "one_launch"])
def test_lists(kind, tpa, precision):
    if kind == "slab":
        s = slab(24, 22, 12, 6.0, 51)
    elif kind == "open":   # a few atoms far above an open surface
        s = I.film(24, 22, 12, 0.0, 0.0, 52, noise=0.05)
        s.x[np.nonzero(s.fixed == 0)[0][::997], 2] += 300.0
        s.box_len = s.box_len + np.array([0.0, 0.0, 300.0])
    elif kind == "dilute":     # 4,000 bricks, 512 slots
        s = dimers(400, 400.0, 53)
    elif kind == "one_tile":   # 419 chunks of cells, one tile of atoms
        s = dimers(200, 400.0, 59)
    else:                      # as many chunks as tiles: still rebuilt in one launch
        s = dimers(3000, 120.0, 60)
    print(f"[case] items {kind} n={s.n} tpa={tpa} {precision}", flush=True)
    sim = md.Simulation(s, tpa=tpa, precision=precision)
    sim.md_build_neighbors(force=True)
    st = sim.md_check()
    assert st["overflow"] == 0 and st["sync_timeout"] == 0, st
    assert check_lists(sim, s) >= s.n // 2 * 2


def test_large_slab_sampled():
    """One share per item (a system that fills the chip): rows of a 216k-atom slab."""
    s = slab(60, 60, 30, 4.0, 54)
    print(f"[case] items large slab n={s.n}", flush=True)
    sim = md.Simulation(s, tpa=2)
    sim.md_build_neighbors(force=True)
    assert sim.md_check()["overflow"] == 0
    rows = np.arange(7, s.n, 1013)
    cnt, idx = O.neighbors(s, s.r_list, x=O.wrap(s), rows=rows)
    got = sim.neighbor_sets(only=rows)
    for t, want in enumerate(O.neighbor_sets(cnt, idx)):
        assert got[rows[t]] == want, rows[t]


def test_batch_in_which_some_rebuild():
    reps = [slab(20, 20, 10, 5.0, 55, temperature=4000.0), dimers(300, 300.0, 56), I.bulk(8, seed=57, temperature=50.0),
            dimers(40, 90.0, 58)]
    print(f"[case] items batch {[s.n for s in reps]}", flush=True)

    def run(systems):
        sim = md.Simulation(systems, tpa=2)
        sim.initial_forces()
        sim.md_run(40)
        st = sim.md_check()
        assert not (st["overflow"] or st["nonfinite"] or st["sync_timeout"]), st
        return sim.state(), sim.md_energy()[:, md.MD_NBUILDS]

    both, builds = run(reps)
    assert builds.min() < 3 < builds.max(), builds   # (some replicas rebuild in steps in which others do not)
    for r, s in enumerate(reps):
        alone, nb = run([s])
        assert nb[0] == builds[r]
        for k in ("x", "v", "f", "dF"):
            assert np.array_equal(alone[0][k], both[r][k]), (r, k)


@pytest.mark.parametrize("list_tgt", [0, 64])
@pytest.mark.parametrize("batch", [False, True])
def test_few_blocks_stride_over_the_items(batch, list_tgt, monkeypatch):
    """An eighth of the blocks, that take item after item, of several replicas that rebuild in different
    steps, against a block per share: lists and trajectories bit for bit."""
    reps = [slab(14, 13, 8, 5.0, 61, temperature=4000.0)]
    if batch:
        reps += [dimers(300, 300.0, 62), I.bulk(7, seed=63, temperature=50.0),
                 I.small_film(nx=12, ny=11, nz=6, radius=6.0, gap=0.5, seed=64)]
    out = []
    for few in ("0", "1"):
        monkeypatch.setenv("MD_LIST_PERSISTENT", few)
        print(f"[case] items few={few} {[s.n for s in reps]} list_tgt={list_tgt}", flush=True)
        sim = md.Simulation(reps, tpa=2, xcap=160, list_tgt=list_tgt)
        sim.initial_forces()
        sim.md_run(25)
        st = sim.md_check()
        assert not (st["overflow"] or st["xoverflow"] or st["nonfinite"] or st["sync_timeout"]), st
        rows = [sim.neighbor_sets(r) for r in range(len(reps))]
        out.append((sim.state(), rows, [sim.neighbor_sets(r, cross=True) for r in range(len(reps))], st))
    for state, rows, cross, st in out[1:]:
        assert rows == out[0][1] and cross == out[0][2] and st == out[0][3]
        for r in range(len(reps)):
            for k in ("x", "v", "f", "dF"):
                assert np.array_equal(state[r][k], out[0][0][r][k]), (r, k)
