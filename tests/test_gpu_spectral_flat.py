"""The isolated hybrid correction of patches one cell thick along z against the oracle: in the query's workspace, and
in one of three complex arrays, where their rows of two modes leave room for two fields only and the components are
formed one after the other.  Tolerance as for the other spectral tests: 1e-12 of
the largest magnitude, a few hundred eps."""

import ctypes

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev, to_host

pytestmark = [pytest.mark.gpu, needs_gpu]


def _three_arrays(shape):
    """One array of n0 x n1 x P2 and two of n0 x P1 x P2 points, the twiddles and four tables of each axis."""
    P = [1 << (2 * n - 1).bit_length() for n in shape]
    up = lambda b: (b + 255) // 256 * 256   # noqa: E731
    tables = up(16 * max(P)) + sum(up(32 * p) for p in P)
    w1, w2 = 16 * shape[0] * shape[1] * P[2], 16 * shape[0] * P[1] * P[2]
    return up(tables + up(w1) + up(w2) + w2)


@pytest.mark.parametrize("room", ["query", "three arrays"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (4, 2, 1), (33, 17, 1), (1, 300, 1), (300, 5, 1), (512, 3, 1), (17, 9, 2)])
def test_flat_isolated_hybrid(shape, room):
    from oracle import spectral
    from paper_1103_6031_amd import mgic
    rng = np.random.default_rng(sum(shape))
    f, base = rng.standard_normal(shape), rng.standard_normal((3,) + shape)
    note("flat isolated hybrid %s, %s" % (shape, room))
    need = mgic.spec_workspace_bytes(shape, isolated=True)
    size = need if room == "query" else _three_arrays(shape)
    assert size <= need
    ws, dims, st = mgic.Workspace(size), (ctypes.c_int * 3)(*shape), mgic._stream()
    out = [to_dev(b) for b in base]
    for k in range(2):                            # the workspace of the first call serves the second
        op, keep = mgic._ptr_array([o.data_ptr() for o in out])
        d = to_dev(f)
        assert mgic._lib.lpt_hybrid_correction(dims, 0.37, 1, 4, 6, -1.3, ctypes.c_void_p(d.data_ptr()), op,
                                               ctypes.c_void_p(ws.ptr), size, st) == mgic.MG_OK
    assert mgic._lib.lpt_hybrid_correction(dims, 0.37, 1, 4, 6, -1.3, ctypes.c_void_p(d.data_ptr()), op,
                                           ctypes.c_void_p(ws.ptr), _three_arrays(shape) - 256, st) == mgic.MG_EINVAL
    corr = spectral.hybrid_correction(f, 0.37, 4, 6, -1.3, periodic=False)
    for c in range(3):
        got = to_host(out[c]) - base[c]
        scale = max(np.max(np.abs(corr[c])), np.max(np.abs(base[c])))
        assert np.max(np.abs(got - 2 * corr[c])) <= 2e-12 * scale
