"""Batches whose depths run by different kernels: a depth of many levels by one-step launches and sweeps, the
depth above it, where only the small instances have a level that the fused tile launches take, by those.

Ten instances of 192^3 have 48^3 levels at depth 2 (2160 tiles with the small instance's: not fused), one of 64^3
its 32^3 level at depth 1 (64 tiles: fused).  Every level's step 6 must run exactly once whatever runs the level
above it, and an instance's bits are those of its solo solve.
"""

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]

SIZES = [64] + [192] * 10


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("nu", [(2, 2), (1, 2)])
def test_a_fused_depth_above_one_that_is_not(prec, nu):
    import torch
    from paper_1103_6031_amd import mgic
    f = {n: to_dev(np.random.default_rng(n).standard_normal((n,) * 3)) for n in set(SIZES)}
    o = mgic.make_opts(prec=prec, fixed_cycles=True, max_cycles=2, nu1=nu[0], nu2=nu[1])
    note("batch depths %s nu=%s" % (prec, nu))
    got, _ = mgic.mg_solve_batch([f[n] for n in SIZES], [100.0 / n for n in SIZES], opts=o)
    for n in f:
        want, _ = mgic.mg_solve_level(f[n], 100.0 / n, opts=o)
        for m, u in zip(SIZES, got):
            assert m != n or torch.equal(u, want), n
