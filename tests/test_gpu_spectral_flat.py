"""The isolated hybrid correction of patches one cell thick along z, whose components are formed one after the other
(rows of two modes leave room for two fields), against the oracle.  Tolerance as for the other spectral tests: 1e-12 of
the largest magnitude, a few hundred eps."""

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev, to_host

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("shape", [(1, 1, 1), (4, 2, 1), (33, 17, 1), (1, 300, 1), (300, 5, 1), (512, 3, 1), (17, 9, 2)])
def test_flat_isolated_hybrid(shape):
    from oracle import spectral
    from paper_1103_6031_amd import mgic
    rng = np.random.default_rng(sum(shape))
    f, base = rng.standard_normal(shape), rng.standard_normal((3,) + shape)
    note("flat isolated hybrid %s" % (shape,))
    ws = mgic.Workspace(mgic.spec_workspace_bytes(shape, isolated=True))
    out = [to_dev(b) for b in base]
    for k in range(2):                            # the workspace of the first call serves the second
        mgic.lpt_hybrid_correction(to_dev(f), 0.37, out, isolated=True, lap_order=4, grad_order=6, scale=-1.3,
                                   workspace=ws)
    corr = spectral.hybrid_correction(f, 0.37, 4, 6, -1.3, periodic=False)
    for c in range(3):
        got = to_host(out[c]) - base[c]
        scale = max(np.max(np.abs(corr[c])), np.max(np.abs(base[c])))
        assert np.max(np.abs(got - 2 * corr[c])) <= 2e-12 * scale
