"""Two red-black sweeps in one launch (periodic power-of-two levels of 128^3 and up) against the one-step
launches: a batched solve smooths every level by half-sweeps, a solo solve these levels by the fused
launch, with the operations on every value in the same order, so the bits are the same.

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
