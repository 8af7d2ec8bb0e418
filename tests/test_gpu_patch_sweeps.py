"""Two sweeps of a patch in one launch, ghost zones formed on the chip, against ghost fills and half-sweeps one
by one, which a workspace without room for the second arrays falls back to: the operations on every value are
in the same order, so the bits are the same.

The patches end inside a tile, are thinner than a tile's halo, span several tiles in every direction, lie in
a patch, and touch the periodic base's boundary.
"""

import ctypes

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]

HIERS = [
    (32, [((16, 16, 32), (4, 5, 6))]),
    (32, [((18, 34, 40), (2, 3, 4))]),
    (32, [((4, 6, 8), (9, 10, 11))]),
    (32, [((20, 24, 48), (3, 2, 1)), ((22, 16, 64), (4, 4, 5))]),
    (64, [((80, 44, 72), (3, 7, 11)), ((48, 40, 64), (6, 4, 5)), ((36, 50, 24), (5, 6, 7))]),
    (32, [((32, 16, 16), (0, 24, 24))]),    # ghosts from the periodic base's other side
    (48, [((64, 66, 36), (5, 6, 7))]),      # rows of 18 cells per colour: half-sweeps in FP32
]


def _small(mgic, hier, fs, o, us=None):
    import torch
    need = mgic.mg_workspace_bytes(hier, o)
    ws, st = mgic.Workspace(need), mgic.mg_stats()
    out = [torch.empty_like(f) for f in fs] if us is None else [u.clone() for u in us]
    fp, keep_f = mgic._ptr_array([f.data_ptr() for f in fs])
    up, keep_u = mgic._ptr_array([u.data_ptr() for u in out])
    H = hier.c_struct()
    rc = mgic._lib.mg_solve_hierarchy(ctypes.byref(H), fp, up, ctypes.byref(o), ctypes.byref(st),
                                      ctypes.c_void_p(ws.ptr), need - 4096, mgic._stream())
    assert rc == mgic.MG_OK
    return out


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("case", range(len(HIERS)))
def test_patch_sweeps_match_the_half_sweeps(case, prec):
    import torch
    from paper_1103_6031_amd import mgic
    n, patches = HIERS[case]
    hier = mgic.Hier(n, 100.0 / n, patches)
    fs = [to_dev(np.random.default_rng(10 * case + p).standard_normal(hier.dims(p))) for p in range(hier.nlev)]
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=3)
    note("patch sweeps: case %d %s, one by one" % (case, prec))
    want = _small(mgic, hier, fs, o)
    note("patch sweeps: case %d %s" % (case, prec))
    for graph in (False, True, True):
        got, _ = mgic.mg_solve_hierarchy(hier, fs, opts=mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=3,
                                                                       graph=graph))
        for a, b in zip(got, want):
            assert torch.equal(a, b)


def test_warm_start():
    import torch
    from paper_1103_6031_amd import mgic
    n, patches = HIERS[3]
    hier = mgic.Hier(n, 100.0 / n, patches)
    rng = np.random.default_rng(5)
    fs, us = ([to_dev(rng.standard_normal(hier.dims(p))) for p in range(hier.nlev)] for _ in range(2))
    o = mgic.make_opts(fixed_cycles=True, max_cycles=2, initial_guess=True)
    note("patch sweeps: warm start")
    want = _small(mgic, hier, fs, o, us)
    got, _ = mgic.mg_solve_hierarchy(hier, fs, u=[u.clone() for u in us], opts=o)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
