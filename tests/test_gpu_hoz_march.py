"""The marched half-sweep of large higher-order patches (2^21 cells and up) against the oracle: sizes whose last
tiles overlap the ones before them in every direction.  After a V-cycle every level of the iterate equals the
oracle's within 1e-12 of its largest value (the two differ in summation order only)."""

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev, to_host
from oracle import zoom, zoom_ho

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("order,n", [(4, (132, 130, 138)), (6, (130, 132, 134)), (2, (162, 164, 166))])
def test_large_patch_matches_the_oracle(order, n):
    from paper_1103_6031_amd import mgic
    N0, patches = 128, [(n, (20, 21, 22))]
    H = zoom.Hierarchy(N0, 100.0 / N0, patches)
    f = [np.random.default_rng(order + p).standard_normal(m) for p, m in enumerate(H.n)]
    note("marched half-sweep: order %d, GPU" % order)
    ug, _ = mgic.mg_solve_hierarchy_ho(mgic.Hier(N0, 100.0 / N0, patches), order, [to_dev(a) for a in f],
                                       opts=mgic.make_opts(max_cycles=1, fixed_cycles=True))
    note("marched half-sweep: order %d, oracle" % order)
    uo, _ = zoom_ho.solve_hierarchy(H, f, order, tol=0.0, max_cycles=1)
    for p in range(2):
        assert np.max(np.abs(to_host(ug[p]) - uo[p])) <= 1e-12 * np.max(np.abs(uo[p]))
