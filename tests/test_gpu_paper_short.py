"""The paper's form with a short cutoff, whose passes take 2 or 4 lanes per atom by the size of the whole
batch: forces against the oracle, and a batch whose replicas take 4 lanes alone and 2 together, bit for
bit."""
import numpy as np
import pytest

import oracle as O
from paper_1507_07068_amd import inputs as I
from paper_1507_07068_amd import md
from tests.test_gpu_parity import FP64_TOL, MIXED_TOL, assert_forces, force_errors

pytestmark = pytest.mark.gpu


def short(s, rc=3.6):
    """Lists of 14 to 26 entries (r_e as in the full form: few entries are expected of it)."""
    s.potential = "paper"
    s.paper["rc"], s.paper["d"] = rc, rc / s.paper["re"]
    s.dt = 0.25
    return s


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("tpa", [1, 2, 4, 8])
@pytest.mark.parametrize("beta", [6.0, 5.0])
def test_forces(precision, tpa, beta):
    s = short(I.small_film(nx=12, ny=11, nz=8, radius=6.0, gap=0.5, seed=81, noise=0.04))
    s.paper["beta"] = beta
    print(f"[case] short lists n={s.n} {precision} tpa={tpa} beta={beta}", flush=True)
    sim = md.Simulation(s, precision=precision, cap=64, xcap=160, tpa=tpa)
    sim.initial_forces()
    st = sim.md_check()
    assert not (st["overflow"] or st["xoverflow"] or st["nonfinite"]), st
    ref = O.evaluate(s, O.wrap(s))
    f = sim.state()[0]["f"]
    if precision == "fp64":
        assert_forces(f, ref["f"], FP64_TOL)
    else:
        assert force_errors(f, ref["f"])[0] <= MIXED_TOL


@pytest.mark.parametrize("precision,shadow", [("fp64", None), ("mixed", True), ("mixed", False)])
@pytest.mark.parametrize("tpa", [1, 2])
def test_lanes_of_a_batch_do_not_show(precision, shadow, tpa):
    reps = [short(I.small_film(nx=28 + 2 * r, ny=25, nz=20 - 4 * r, radius=8.0, gap=0.3, seed=82 + r, noise=0.03))
            for r in range(2)]
    print(f"[case] short lists {[s.n for s in reps]} {precision} shadow={shadow} tpa={tpa}", flush=True)
    assert max(s.n for s in reps) < 49152 - 512 and sum(s.n for s in reps) > 49152

    def run(systems):
        sim = md.Simulation(systems, precision=precision, cap=64, xcap=160, tpa=tpa, shadow=shadow)
        sim.initial_forces()
        sim.md_run(8)
        return sim.state()

    both = run(reps)
    for r, s in enumerate(reps):
        alone = run([s])[0]
        for k in ("x", "v", "f", "dF"):
            assert np.array_equal(alone[k], both[r][k]), (r, k)
