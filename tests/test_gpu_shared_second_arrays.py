"""Swept levels whose second array is the first u of the level above: hierarchies with patches no smaller than their
parents, and bases whose coarsenings are swept too, against the half-sweeps that a workspace without room for the
second arrays runs (the same operations in the same order: the same bits).  Converging solves, so that every cycle
and every outer step follows the ones before.
"""

import ctypes

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]

HIERS = [
    (48, [((48, 48, 48), (5, 6, 7)), ((64, 64, 64), (6, 7, 8))]),     # each array the one above's, down to 48^3
    (160, [((48, 64, 56), (50, 40, 30)), ((64, 80, 72), (5, 4, 6))]),  # the base larger than its patch
    (160, []),
    (192, [((192, 192, 192), (40, 50, 48))]),                          # 192^3, the base and its 96^3
]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("case", range(len(HIERS)))
def test_shared_arrays_match_the_half_sweeps(case, prec):
    import torch
    from paper_1103_6031_amd import mgic
    n, patches = HIERS[case]
    hier = mgic.Hier(n, 100.0 / n, patches)
    fs = [to_dev(np.random.default_rng(20 * case + p).standard_normal(hier.dims(p))) for p in range(hier.nlev)]
    o = mgic.make_opts(prec=prec, tol=1e-9, max_cycles=40)
    need = mgic.mg_workspace_bytes(hier, o)
    ws, st = mgic.Workspace(need), mgic.mg_stats()
    want = [torch.empty_like(f) for f in fs]
    fp, keep_f = mgic._ptr_array([f.data_ptr() for f in fs])
    up, keep_u = mgic._ptr_array([u.data_ptr() for u in want])
    H = hier.c_struct()
    note("shared second arrays: case %d %s, one by one" % (case, prec))
    rc = mgic._lib.mg_solve_hierarchy(ctypes.byref(H), fp, up, ctypes.byref(o), ctypes.byref(st),
                                      ctypes.c_void_p(ws.ptr), need - 4096, mgic._stream())
    assert rc == mgic.MG_OK
    note("shared second arrays: case %d %s" % (case, prec))
    for _ in range(3):
        got, stats = mgic.mg_solve_hierarchy(hier, fs, opts=o, workspace=ws)
        assert stats["cycles"] == st.cycles
        for a, b in zip(got, want):
            assert torch.equal(a, b)


def test_more_room_than_the_query_asks_for_gives_every_second_array():
    """FP64 160^3: with a second u of the finest level the plan would pass the static scratch array, so the query
    leaves it out and the finest level takes half-sweeps; a workspace with room for it takes two sweeps a launch."""
    import torch
    from paper_1103_6031_amd import mgic
    n, cycles = 160, 3
    f = to_dev(np.random.default_rng(3).standard_normal((n,) * 3))
    o = mgic.make_opts(fixed_cycles=True, max_cycles=cycles)
    need = mgic.mg_workspace_bytes(mgic.Hier(n, 1.0), o)
    got, launches = [], []
    for room in (0, 8 * n ** 3 + 4096):
        note("more room than the query: %d" % room)
        mgic.mg_kprof_enable(1)
        got.append(mgic.mg_solve_level(f, 1.0, opts=o, workspace=mgic.Workspace(need + room))[0])
        launches.append(mgic.mg_kprof_read()[1])
        mgic.mg_kprof_enable(0)
    assert launches == [8 * cycles, 2 * cycles]
    assert torch.equal(got[0], got[1])
    note("more room than the query: batch")
    ws = mgic.Workspace(mgic.mg_batch_workspace_bytes([n, n], o) + 2 * (8 * n ** 3 + 4096))
    for u in mgic.mg_solve_batch([f, f], [1.0, 1.0], opts=o, workspace=ws)[0]:
        assert torch.equal(u, got[0])
