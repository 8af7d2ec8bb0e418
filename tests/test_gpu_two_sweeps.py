"""Two red-black sweeps in one launch against the one-step launches, which a batch workspace without room for
the second arrays takes at every level: the operations on every value are in the same order, so the bits are
the same.  A solo solve and a batched one choose different tiles.

256^3 marches in blocks of 32 planes over several tiles in y and z and has a fused 128^3 coarsening
(blocks of 8 planes); mixed solves start from the red half-sweep of the outer step, every cycle ends with
the correction added to the black cells; three cycles carry the result of each through the others.
"""

import ctypes

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]


def _f(n, seed=0):
    return np.random.default_rng(n + seed).standard_normal((n,) * 3)


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("n", [128, 256])
def test_two_sweeps_match_the_half_sweeps(n, prec):
    import torch
    from paper_1103_6031_amd import mgic
    f = to_dev(_f(n))
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=6)
    note("two sweeps n=%d %s" % (n, prec))
    want, _ = mgic.mg_solve_batch([f], [100.0 / n], opts=o)
    for graph in (False, True, True, True):
        got, _ = mgic.mg_solve_level(f, 100.0 / n, opts=mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=6,
                                                                       graph=graph))
        assert torch.equal(got, want[0])


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_initial_guess_and_small_workspace(prec):
    """A warm start, and a workspace without room for the second arrays (half-sweep launches)."""
    import torch
    from paper_1103_6031_amd import mgic
    n, h = 128, 100.0 / 128
    f, g = to_dev(_f(n, 1)), to_dev(_f(n, 2))
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=2, initial_guess=True)
    want, _ = mgic.mg_solve_batch([f], [h], u=[g.clone()], opts=o)
    note("two sweeps: warm start %s" % prec)
    got, _ = mgic.mg_solve_level(f, h, u=g.clone(), opts=o)
    assert torch.equal(got, want[0])
    need = mgic.mg_workspace_bytes(mgic.Hier(n, h), o)
    ws, u, st = mgic.Workspace(need), g.clone(), mgic.mg_stats()
    rc = mgic._lib.mg_solve_level(n, h, f.data_ptr(), u.data_ptr(), ctypes.byref(o), ctypes.byref(st),
                                  ctypes.c_void_p(ws.ptr), need - 4096, mgic._stream())
    assert rc == mgic.MG_OK and torch.equal(u, want[0])


# tiles that overlap at the level's edge in every direction, levels of one tile, odd counts of 16-byte runs;
# the last two are 4 x odd cells wide (half-sweeps in FP32: rows of a colour are no whole runs)
SIZES = [32, 40, 48, 56, 80, 96, 112, 128, 160, 192, 224, 20, 28]


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_every_level_size_matches_the_half_sweeps(prec):
    import torch
    from paper_1103_6031_amd import mgic
    fs = [to_dev(_f(n, 11)) for n in SIZES]
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=3)
    need = mgic.mg_batch_workspace_bytes(SIZES, o)
    ws = mgic.Workspace(need)
    note("two sweeps: half-sweep batch %s" % prec)
    n = (ctypes.c_int * len(SIZES))(*SIZES)
    h = (ctypes.c_double * len(SIZES))(*[100.0 / v for v in SIZES])
    want = [torch.empty_like(f) for f in fs]
    fp, keep_f = mgic._ptr_array([f.data_ptr() for f in fs])
    up, keep_u = mgic._ptr_array([u.data_ptr() for u in want])
    st = (mgic.mg_stats * len(SIZES))()
    rc = mgic._lib.mg_solve_batch(len(SIZES), n, h, fp, up, ctypes.byref(o), st, ctypes.c_void_p(ws.ptr),
                                  need - 4096, mgic._stream())
    assert rc == mgic.MG_OK
    note("two sweeps: batch %s" % prec)
    got, _ = mgic.mg_solve_batch(fs, [100.0 / v for v in SIZES], opts=o, workspace=ws)
    for v, f, a, b in zip(SIZES, fs, want, got):
        assert torch.equal(a, b), v
        note("two sweeps: solo %d %s" % (v, prec))
        solo, _ = mgic.mg_solve_level(f, 100.0 / v, opts=o)
        assert torch.equal(a, solo), v


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("n", [48, 80, 96])
def test_base_under_a_patch(n, prec):
    """The base of a hierarchy: the second array is its own, the sweeps start from both colours' values."""
    import torch
    from paper_1103_6031_amd import mgic
    hier = mgic.Hier(n, 100.0 / n, [((32, 24, 16), (5, 8, 11))])
    fs = [to_dev(np.random.default_rng(n + p).standard_normal(hier.dims(p))) for p in range(2)]
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=3)
    note("two sweeps: base %d under a patch, %s" % (n, prec))
    got, _ = mgic.mg_solve_hierarchy(hier, fs, opts=o)
    need = mgic.mg_workspace_bytes(hier, o)
    ws, st = mgic.Workspace(need), mgic.mg_stats()
    want = [torch.empty_like(f) for f in fs]
    fp, keep_f = mgic._ptr_array([f.data_ptr() for f in fs])
    up, keep_u = mgic._ptr_array([u.data_ptr() for u in want])
    H = hier.c_struct()
    rc = mgic._lib.mg_solve_hierarchy(ctypes.byref(H), fp, up, ctypes.byref(o), ctypes.byref(st),
                                      ctypes.c_void_p(ws.ptr), need - 4096, mgic._stream())
    assert rc == mgic.MG_OK
    for a, b in zip(got, want):
        assert torch.equal(a, b)
