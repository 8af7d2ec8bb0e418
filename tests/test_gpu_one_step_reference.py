"""The fused tile launches and the sweeps in one launch against one-step launches, which the smallest workspaces take
at every level: a batch without room for any second array (half a page below its query), and a solo solve in the
plain workspace (half-sweeps above the fused levels).  The operations on every value are in the same order, so the
bits are the same.
"""

import ctypes

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]

# fused levels of 16^3 to 64^3 of every base, tiles that end inside the level, levels above them
SIZES = [24, 32, 40, 56, 64, 80, 96, 112, 128, 160]


def _batch_one_step(mgic, fs, sizes, o):
    import torch
    need = mgic.mg_batch_workspace_bytes(sizes, o)
    ws = mgic.Workspace(need)
    n = (ctypes.c_int * len(sizes))(*sizes)
    h = (ctypes.c_double * len(sizes))(*[100.0 / v for v in sizes])
    out = [torch.empty_like(f) for f in fs]
    fp, keep_f = mgic._ptr_array([f.data_ptr() for f in fs])
    up, keep_u = mgic._ptr_array([u.data_ptr() for u in out])
    st = (mgic.mg_stats * len(sizes))()
    rc = mgic._lib.mg_solve_batch(len(sizes), n, h, fp, up, ctypes.byref(o), st, ctypes.c_void_p(ws.ptr), need - 2048,
                                  mgic._stream())
    assert rc == mgic.MG_OK
    return out


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("nu", [(2, 2), (1, 2), (2, 1), (1, 1)])
def test_fused_levels(prec, nu):
    import torch
    from paper_1103_6031_amd import mgic
    fs = [to_dev(np.random.default_rng(n + 40).standard_normal((n,) * 3)) for n in SIZES]
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=3, nu1=nu[0], nu2=nu[1])
    note("one-step reference: batch %s nu=%s" % (prec, nu))
    want = _batch_one_step(mgic, fs, SIZES, o)
    note("one-step reference: fused batch %s nu=%s" % (prec, nu))
    got, _ = mgic.mg_solve_batch(fs, [100.0 / n for n in SIZES], opts=o)
    for n, f, a, b in zip(SIZES, fs, want, got):
        assert torch.equal(a, b), n
        note("one-step reference: solo %d %s nu=%s" % (n, prec, nu))
        solo, _ = mgic.mg_solve_level(f, 100.0 / n, opts=o)
        assert torch.equal(a, solo), n


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("n", [256, 384, 512])
def test_sweeps_of_large_levels(n, prec):
    """Solo tiles of large levels, the launches counted: two a cycle on the finest level (in mixed precision the
    outer step's half-sweep comes before the first), against eight (seven)."""
    import torch
    from paper_1103_6031_amd import mgic
    g = torch.Generator(device="cuda:0").manual_seed(n)
    f = torch.randn((n,) * 3, generator=g, dtype=torch.float64, device="cuda:0")
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=2)
    hier = mgic.Hier(n, 100.0 / n)
    out, launches = [], []
    for size in (mgic.mg_plain_workspace_bytes, mgic.mg_workspace_bytes):
        note("one-step reference: solo %d %s, %s" % (n, prec, size.__name__))
        ws = mgic.Workspace(size(hier, o))
        mgic.mg_kprof_enable(1)
        out.append(mgic.mg_solve_level(f, 100.0 / n, opts=o, workspace=ws)[0])
        launches.append(mgic.mg_kprof_read()[1])
        mgic.mg_kprof_enable(0)
    assert torch.equal(out[0], out[1])
    assert launches[1] == 4 and launches[0] >= 13
