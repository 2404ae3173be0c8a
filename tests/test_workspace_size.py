"""Workspace sizes of two-tier lists (host side): the middle lists are kept where the outer lists are
long and well over their length, and cost no memory where they would not pay."""
import ctypes as C

import pytest

from paper_1507_07068_amd import inputs as I
from paper_1507_07068_amd import md


def workspace(s, cap, icap):
    lib = md.load_library()
    p = md.make_params(s, cap=cap, xcap=64, tpa=2, icap=icap)
    h = C.c_void_p()
    desc = (md.ReplicaDesc * 1)(md.make_replica_desc(s))
    assert lib.md_system_create(C.cast(desc, C.c_void_p), 1, C.byref(p), C.byref(h)) == md.MD_OK
    n = int(lib.md_workspace_bytes(h))
    lib.md_system_destroy(h)
    return n


@pytest.mark.parametrize("potential,skin,cap,icap,kept", [
    ("fs", 0.3, 64, 64, False), ("fs", 0.6, 192, 64, False), ("fs", 2.2, 192, 64, False), ("fs", 2.2, 1024, 64, False),
    ("paper", 0.3, 256, 224, False), ("paper", 0.66, 1152, 256, False), ("paper", 1.5, 384, 256, True),
    ("paper", 5.7834, 1152, 256, True)])
def test_middle_lists(potential, skin, cap, icap, kept):
    s = I.bulk(16, seed=1)
    s.potential, s.skin = potential, skin
    one, two = workspace(s, cap, 0), workspace(s, cap, icap)
    assert (two > one + 4 * icap * s.n) if kept else two <= one + 1024
