"""A red-black sweep of the higher-order levels in one launch: sizes of one tile and of several, odd sweep
counts (whose last sweep runs as two half-sweeps), and FP32 inner cycles, against the oracle.

After a fixed number of V-cycles the FP64 iterate equals the oracle's within 1e-12 of its largest value
(the two differ in summation order only); the mixed solve is within 1e-8 relative RMS of the exact solution,
as in the other higher-order tests.
"""

import numpy as np
import pytest

from gpu_util import needs_gpu, note, rel_rms, to_dev, to_host
from oracle import highorder as ho

pytestmark = [pytest.mark.gpu, needs_gpu]


def _f(n, order):
    return np.random.default_rng(31 * n + order).standard_normal((n,) * 3)


@pytest.mark.parametrize("order", [2, 4, 6])
@pytest.mark.parametrize("n,nu", [(64, (2, 2)), (128, (2, 2)), (64, (3, 2)), (128, (2, 1)), (32, (4, 2))])
def test_sweeps_match_the_oracle(order, n, nu):
    from paper_1103_6031_amd import mgic
    f, h = _f(n, order), 50.0 / n
    note("ho sweep order %d n=%d nu=%s" % (order, n, nu))
    ug, _ = mgic.mg_solve_level_ho(to_dev(f), h, order, opts=mgic.make_opts(max_cycles=1, fixed_cycles=True,
                                                                            nu1=nu[0], nu2=nu[1]))
    uo, _ = ho.solve_level(f, h, order, max_cycles=1, fixed_cycles=True, nu1=nu[0], nu2=nu[1])
    assert np.max(np.abs(to_host(ug) - uo)) <= 1e-12 * np.max(np.abs(uo))


@pytest.mark.parametrize("order", [2, 4, 6])
@pytest.mark.parametrize("n", [64, 128])
def test_mixed_precision(order, n):
    from paper_1103_6031_amd import mgic
    f, h = _f(n, order), 50.0 / n
    note("ho sweep mixed order %d n=%d" % (order, n))
    o = mgic.make_opts(tol=1e-10, prec="mixed")
    um, _ = mgic.mg_solve_level_ho(to_dev(f), h, order, opts=o)
    ud, _ = mgic.mg_solve_level_ho(to_dev(f), h, order, opts=mgic.make_opts(tol=1e-12))
    assert rel_rms(to_host(um), to_host(ud)) <= 1e-8
