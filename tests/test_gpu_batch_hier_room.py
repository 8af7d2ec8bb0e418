"""A hierarchy batch in a workspace without room for the second arrays: every part runs without them, same bits."""

import ctypes

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]

# instances with one and two patches, bases in and outside the batched schedule
SHAPES = [(64, [((64, 64, 64), (16, 16, 16)), ((48, 64, 56), (10, 8, 9))]), (32, [((16, 16, 32), (4, 5, 6))]),
          (48, []), (64, []), (16, [])]
# what the plans without second arrays take
PLAIN = {"fp64": 22790144, "mixed": 37410816}


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_a_workspace_of_the_plain_plans_is_taken(prec):
    import torch
    from paper_1103_6031_amd import mgic
    hs = [mgic.Hier(n, 100.0 / n, p) for n, p in SHAPES]
    fs = [[to_dev(np.random.default_rng(7 * i + p).standard_normal(h.dims(p))) for p in range(h.nlev)]
          for i, h in enumerate(hs)]
    o = mgic.make_opts(prec=prec, tol=1e-9, max_cycles=40)
    assert mgic.mg_batch_hier_workspace_bytes(hs, o) > PLAIN[prec]
    note("hierarchy batch, full workspace, %s" % prec)
    want, _ = mgic.mg_solve_batch_hier(hs, fs, opts=o)
    got = [[torch.empty_like(x) for x in f] for f in fs]
    hp, _keep = mgic._hier_array(hs)
    fl = [mgic._ptr_array([x.data_ptr() for x in f]) for f in fs]
    ul = [mgic._ptr_array([x.data_ptr() for x in u]) for u in got]
    fa = (mgic._PP * len(hs))(*[p for p, _ in fl])
    ua = (mgic._PP * len(hs))(*[p for p, _ in ul])
    st = (mgic.mg_stats * len(hs))()
    ws = mgic.Workspace(PLAIN[prec])

    def call(room):
        return mgic._lib.mg_solve_batch_hier(len(hs), hp, ctypes.cast(fa, ctypes.c_void_p),
                                             ctypes.cast(ua, ctypes.c_void_p), ctypes.byref(o), st,
                                             ctypes.c_void_p(ws.ptr), room, mgic._stream())

    note("hierarchy batch, plain workspace, %s" % prec)
    assert call(PLAIN[prec]) == mgic.MG_OK
    for a, b in zip(got, want):
        for x, y in zip(a, b):
            assert torch.equal(x, y)
    assert call(PLAIN[prec] // 2) == mgic.MG_EINVAL and b"too small" in mgic._lib.mg_last_error()
