"""The middle list of two-tier lists: inner lists taken from it are those taken from the outer
list, so a run with a workspace that holds it and one with the static scratch, which here does
not, agree bit for bit."""
import numpy as np
import pytest

from paper_1507_07068_amd import inputs as I
from paper_1507_07068_amd import md

pytestmark = pytest.mark.gpu


# icap 208: the middle lists hold 264 entries, 258 being a lattice atom's, so that with the
# thermal motion some atoms fall back to the outer list; 256: 328, and all fit
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("icap,tpa", [(208, 2), (256, 1), (256, 8)])
def test_runs_agree_with_and_without(icap, tpa, precision):
    s = I.two_tier(I.film(22, 22, 18, 8.0, 0.5, 91, noise=0.02, temperature=2000.0))
    print(f"[case] middle list n={s.n} icap={icap} tpa={tpa} {precision}", flush=True)
    sims = [md.Simulation(s, precision=precision, cap=1152, xcap=160, tpa=tpa, icap=icap, static_workspace=st)
            for st in (False, True)]
    # the middle lists alone would take more than the static scratch
    assert 4 * s.n * (icap + 56) >= md.MD_SCRATCH_BYTES
    for m in sims:
        m.initial_forces()
    for steps in (1, 40, 60):
        for m in sims:
            m.run(steps)
        a, b = (m.state()[0] for m in sims)
        for k in ("x", "v", "f", "dF"):
            assert np.array_equal(a[k], b[k]), (steps, k)
        ia, ib = (m.neighbor_sets(0, only=range(0, s.n, 37), inner=True) for m in sims)
        assert ia == ib
    assert np.abs(a["x"] - s.x).max() > 0.35   # past half the middle skin: it was taken again
    st = [m.md_check() for m in sims]
    assert all(t["overflow"] == 0 and t["ioverflow"] == 0 and t["nonfinite"] == 0 for t in st), st
