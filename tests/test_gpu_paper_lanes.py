"""The paper form's passes: lanes per atom and the power of its density function.

The passes take 4 or 8 lanes per atom by the size of the whole batch, with sums that agree bit
for bit, and f(r) = fe (re / r)^beta by products when beta / 2 is a whole number 1..8, else
through pow."""
import numpy as np
import pytest

import oracle as O
from paper_1507_07068_amd import inputs as I
from paper_1507_07068_amd import md
from tests.test_gpu_parity import FP64_TOL, assert_forces
from tests.test_gpu_parity_paper import CAP, initial, paper, psim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,shadow", [("fp64", None), ("mixed", True), ("mixed", False)])
@pytest.mark.parametrize("tpa", [1, 4])
def test_lanes_of_a_batch_do_not_show(precision, shadow, tpa):
    """Two films of 28,000 and 24,300 atoms: 8 lanes per atom each alone, 4 together."""
    reps = [paper(I.small_film(nx=28 + 2 * r, ny=25, nz=20 - 4 * r, radius=8.0, gap=0.3, seed=80 + r, noise=0.03))
            for r in range(2)]
    print(f"[case] paper lanes {[s.n for s in reps]} {precision} shadow={shadow} tpa={tpa}", flush=True)
    assert max(s.n for s in reps) < 49152 - 512 and sum(s.n for s in reps) > 49152
    b = md.Simulation(reps, precision=precision, cap=CAP, xcap=160, tpa=tpa, shadow=shadow)
    b.initial_forces()
    b.run(6)
    stb = b.state()
    for r, s in enumerate(reps):
        a = psim(s, precision=precision, tpa=tpa, shadow=shadow)
        a.initial_forces()
        a.run(6)
        sta = a.state()[0]
        for k in ("x", "v", "f", "dF"):
            assert np.array_equal(sta[k], stb[r][k]), (r, k)


@pytest.mark.parametrize("beta", [2.0, 4.0, 5.0, 6.5, 8.0, 10.0, 14.0, 16.0, 18.0])
def test_density_power(beta):
    """Both sides of the rule (whole beta / 2 up to 8, else pow) against the oracle's pow: the
    products differ from it by a few ulp."""
    s = paper(I.bulk(8, seed=70, noise=0.05, name=f"paper_beta{beta}"))
    s.paper["beta"] = beta
    sim = psim(s, tpa=2)
    _, st = initial(sim)
    ref = O.evaluate(s, O.wrap(s))
    assert np.allclose(st["rho"], ref["rho"], rtol=1e-12, atol=0)
    assert_forces(st["f"], ref["f"], FP64_TOL)
