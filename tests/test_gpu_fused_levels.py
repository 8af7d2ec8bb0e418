"""The fused tile launches of coarsenings that are no power of two, against the one-step launches.

A batched solve runs every level by one-step launches, a solo solve the levels of 20 .. 56 cells by
the fused ones (tiles of 8 that end inside the level at 20 and 28): the same operations in the same
order, so the same bits.  Bases of 3, 5 and 7 times a power of two also end in the three coarsest
solvers; their converged solution is the FFT solution of the same stencil, within the solve's
tolerance 1e-12 times the condition of the discrete Poisson problem's smoothest mode (the residual
norm bounds that mode's error one to one, so 1e-9 of the largest value is ample).
"""

import ctypes

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev, to_host

pytestmark = [pytest.mark.gpu, needs_gpu]

SIZES = [24, 40, 56, 80, 96, 112, 160]


def _f(n, seed=0):
    return np.random.default_rng(n + seed).standard_normal((n,) * 3)


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("nu", [(2, 2), (1, 2), (1, 1)])
def test_fused_levels_match_the_one_step_launches(prec, nu):
    import torch
    from paper_1103_6031_amd import mgic
    fs, hs = [to_dev(_f(n)) for n in SIZES], [100.0 / n for n in SIZES]
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=3, nu1=nu[0], nu2=nu[1])
    note("fused levels %s nu=%s" % (prec, nu))
    ub, _ = mgic.mg_solve_batch(fs, hs, opts=o)
    for n, f, h, u in zip(SIZES, fs, hs, ub):
        solo, _ = mgic.mg_solve_level(f, h, opts=o)
        assert torch.equal(solo, u), n


@pytest.mark.parametrize("n", [24, 40, 56, 112])
def test_converged_solution_is_the_fft_solution(n):
    from oracle import periodic
    from paper_1103_6031_amd import mgic
    f, h = _f(n, 7), 100.0 / n
    note("fused levels: converged n=%d" % n)
    u, st = mgic.mg_solve_level(to_dev(f), h, opts=mgic.make_opts(tol=1e-12, max_cycles=40))
    want = periodic.fft_solve(f - f.mean(), h)
    assert np.max(np.abs(to_host(u) - want)) <= 1e-9 * np.max(np.abs(want))
    assert st["cycles"] <= 16


def test_workspace_without_the_second_arrays():
    """A workspace too small for the fused arrays of 48^3 and 24^3 runs those levels one by one."""
    import torch
    from paper_1103_6031_amd import mgic
    n, h = 96, 100.0 / 96
    f = to_dev(_f(n, 3))
    o = mgic.make_opts(prec="fp64", fixed_cycles=True, max_cycles=2)
    want, _ = mgic.mg_solve_level(f, h, opts=o)
    need = mgic.mg_workspace_bytes(mgic.Hier(n, h), o)
    ws, u, st = mgic.Workspace(need), torch.empty_like(f), mgic.mg_stats()
    note("fused levels: small workspace")
    rc = mgic._lib.mg_solve_level(n, h, f.data_ptr(), u.data_ptr(), ctypes.byref(o), ctypes.byref(st),
                                  ctypes.c_void_p(ws.ptr), need - 8 * 2 * 24 ** 3, mgic._stream())
    assert rc == mgic.MG_OK and torch.equal(u, want)
    rc = mgic._lib.mg_solve_level(n, h, f.data_ptr(), u.data_ptr(), ctypes.byref(o), ctypes.byref(st),
                                  ctypes.c_void_p(ws.ptr), need // 2, mgic._stream())
    assert rc == mgic.MG_EINVAL


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_batched_fused_levels_match_their_one_step_launches(prec):
    """A batch workspace without room for the second arrays runs every level by one-step launches."""
    import torch
    from paper_1103_6031_amd import mgic
    sizes = [32, 24, 64, 40, 112, 256, 96]
    fs = [to_dev(_f(n, 5)) for n in sizes]
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=2)
    need = mgic.mg_batch_workspace_bytes(sizes, o)
    ws = mgic.Workspace(need)
    note("batched fused levels %s" % prec)
    want, _ = mgic.mg_solve_batch(fs, [100.0 / n for n in sizes], opts=o, workspace=ws)
    n = (ctypes.c_int * len(sizes))(*sizes)
    h = (ctypes.c_double * len(sizes))(*[100.0 / v for v in sizes])
    got = [torch.empty_like(f) for f in fs]
    fp, keep_f = mgic._ptr_array([f.data_ptr() for f in fs])
    up, keep_u = mgic._ptr_array([u.data_ptr() for u in got])
    st = (mgic.mg_stats * len(sizes))()
    rc = mgic._lib.mg_solve_batch(len(sizes), n, h, fp, up, ctypes.byref(o), st, ctypes.c_void_p(ws.ptr),
                                  need - 4096, mgic._stream())
    assert rc == mgic.MG_OK
    for a, b in zip(got, want):
        assert torch.equal(a, b)
