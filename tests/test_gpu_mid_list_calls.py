"""Two-tier lists over several calls: the inner lists of a call are taken from the outer lists that
the call is given, whatever was given to the call before (arrays changed in place, other arrays,
arrays put back), and in a batch each replica's are its own (one replica outruns its middle lists,
the other keeps them)."""
import numpy as np
import pytest

from paper_1507_07068_amd import inputs as I
from paper_1507_07068_amd import md
from tests.test_gpu_parity import min_image_diff

pytestmark = pytest.mark.gpu


def check_inner_of_outer(sim, s):
    """Every inner list is the outer list's entries closer than the cutoff, in their order."""
    q = sim.q.cpu().numpy()
    rows = range(0, s.n, 23)
    kept = 0
    for p, outer, inner in zip(rows, sim.list_rows(rows), sim.list_rows(rows, inner=True)):
        d = q[outer, :3] - q[p, :3]
        for a in range(3):
            if s.periodic[a]:
                d[:, a] -= s.box_len[a] * np.round(d[:, a] / s.box_len[a])
        r2 = (d * d).sum(1)
        assert np.abs(r2 - s.cutoff ** 2).min(initial=1.0) > 1e-9   # (no pair for rounding to decide)
        assert np.array_equal(inner, outer[r2 < s.cutoff ** 2]), p
        kept += len(inner)
    st = sim.md_check()
    assert not (st["overflow"] or st["ioverflow"] or st["nonfinite"]), st
    return kept


@pytest.mark.parametrize("how", ["calls", "run", "graph"])
@pytest.mark.parametrize("tpa", [1, 4])
def test_outer_lists_changed_between_calls(how, tpa):
    import torch
    s = I.two_tier(I.bulk(16, seed=71, noise=0.03, temperature=10.0))
    print(f"[case] changed outer lists n={s.n} {how} tpa={tpa}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim = md.Simulation(s, cap=1152, tpa=tpa, icap=256)
        sim.initial_forces()
        graph = sim.md_graph_create(2) if how == "graph" else None

        def go():
            if how == "graph":
                sim.md_graph_launch(graph)
            elif how == "run":
                sim.md_run(2)
            else:
                sim.md_eam_forces(md.MD_F_DENSITY | md.MD_F_FORCE)
            return check_inner_of_outer(sim, s)

        whole = go()
        idx0, cnt0 = sim.idx.clone(), sim.cnt.clone()
        sim.cnt -= sim.cnt // 2                  # fewer entries
        assert go() < 0.7 * whole
        sim.cnt.copy_(cnt0)                      # put back
        assert abs(go() - whole) < 0.01 * whole
        # other entries, as many: the words of a stride in reverse order, within each atom's own
        # first entries (a multiple of tpa that every list has)
        m = int(cnt0[:s.n].min()) // tpa * tpa
        w = sim.idx.view(-1, sim.ntot, tpa)
        w[:m // tpa] = w[:m // tpa].flip(0)
        assert abs(go() - whole) < 0.01 * whole
        sim.idx.copy_(idx0)
        go()
        if how != "graph":                       # other arrays
            sim.idx, sim.cnt, sim._lists_c = idx0.clone(), cnt0 - cnt0 // 2, None
            assert go() < 0.7 * whole
        assert sim.md_check()["nbuilds"] == 1


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("how", ["run", "graph"])
def test_batch_of_a_fast_and_a_slow_replica(how, precision):
    import torch
    reps = [I.two_tier(I.bulk(16, seed=72, noise=0.01, temperature=5.0)),
            I.two_tier(I.bulk(15, seed=73, noise=0.02, temperature=2500.0))]
    print(f"[case] two-tier batch {[s.n for s in reps]} {how} {precision}", flush=True)

    def states(systems):
        stream = torch.cuda.Stream()
        out = []
        with torch.cuda.stream(stream):
            sim = md.Simulation(systems, precision=precision, cap=1152, xcap=160, tpa=2, icap=256)
            sim.initial_forces()
            graph = sim.md_graph_create(30) if how == "graph" else None
            for _ in range(4):
                sim.md_graph_launch(graph) if how == "graph" else sim.md_run(30)
                out.append(sim.state())
            st = sim.md_check()
            assert not (st["overflow"] or st["xoverflow"] or st["ioverflow"] or st["nonfinite"]), st
            assert st["nbuilds"] == len(systems)
        return out

    both = states(reps)
    for r, s in enumerate(reps):
        for alone, batch in zip(states([s]), both):
            for k in ("x", "v", "f", "dF"):
                assert np.array_equal(alone[0][k], batch[r][k]), (r, k)
    moved = [np.abs(min_image_diff(both[-1][r]["x"], s.x, s)).max() for r, s in enumerate(reps)]
    half = 0.5 * 0.08 * reps[0].cutoff   # of the middle lists' own skin
    assert moved[0] < half < 1.2 * half < moved[1], moved


def test_workspace_without_the_middle_lists():
    """The size that the system needs with icap 0 is taken (and gives the same forces), a smaller
    one is refused."""
    import ctypes as C

    import torch
    s = I.two_tier(I.bulk(16, seed=74, noise=0.03, temperature=300.0))
    lib = md.load_library()
    p = md.make_params(s, cap=1152, xcap=160, tpa=2)
    h = C.c_void_p()
    desc = (md.ReplicaDesc * 1)(md.make_replica_desc(s))
    assert lib.md_system_create(C.cast(desc, C.c_void_p), 1, C.byref(p), C.byref(h)) == md.MD_OK
    need = int(lib.md_workspace_bytes(h))
    lib.md_system_destroy(h)
    sims = [md.Simulation(s, cap=1152, xcap=160, tpa=2, icap=256) for _ in range(2)]
    small = sims[1]
    whole = int(lib.md_workspace_bytes(small.handle))
    print(f"[case] workspace {need} of {whole} bytes", flush=True)
    assert need + 4 * 256 * s.n < whole
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert ws.data_ptr() % 256 == 0
    assert lib.md_workspace_bind(small.handle, C.c_void_p(ws.data_ptr()), need - 1, small.stream) == md.MD_ERR_ARG
    small.ws = ws
    assert lib.md_workspace_bind(small.handle, C.c_void_p(ws.data_ptr()), need, small.stream) == md.MD_OK
    for m in sims:
        m.initial_forces()
        m.md_run(20)
    a, b = (m.state()[0] for m in sims)
    for k in ("x", "v", "f", "dF"):
        assert np.array_equal(a[k], b[k]), k
