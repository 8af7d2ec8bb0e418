"""The x-marched LPT tiles (levels of at least 2^21 cells that 16 x 64 tiles divide) against plain 64-bit
torch, with 16-byte aligned arrays and with arrays that start 8 bytes off (loads cell by cell).

128^3 takes the shortest march (8 planes), 192^3 an odd number of tiles along z, 256^3 32 planes.
Tolerance: a G4 value is a sum of four terms of up to 8 max|phi| / (12 h), rounded a few times: some
eps of that; tau and det combine six and nine of them: 1e-12 of the largest magnitude covers both.
"""

import numpy as np
import pytest

from gpu_util import needs_gpu, note

pytestmark = [pytest.mark.gpu, needs_gpu]

TOL = 1e-12


def _dev(t, skew):
    import torch
    buf = torch.empty(t.numel() + skew, dtype=torch.float64, device="cuda:0")
    out = buf[skew:].view(t.shape)
    out.copy_(t)
    return out


def _g4(x, axis, h):
    import torch
    r = lambda s: torch.roll(x, -s, axis)
    return (r(-2) - 8.0 * r(-1) + 8.0 * r(1) - r(2)) / (12.0 * h)


def _close(got, want):
    err, top = float((got - want).abs().max()), float(want.abs().max())
    assert err <= TOL * top, (err, top)


@pytest.mark.parametrize("skew", [0, 1])
@pytest.mark.parametrize("n", [128, 192, 256])
def test_tiles_match_torch(n, skew):
    import torch
    from paper_1103_6031_amd import mgic
    h = 100.0 / n
    H = mgic.Hier(n, h)
    g = torch.Generator(device="cuda:0").manual_seed(n + skew)
    phi = _dev(torch.randn((n,) * 3, generator=g, dtype=torch.float64, device="cuda:0"), skew)
    note("LPT tiles n %d skew %d" % (n, skew))
    out = [[_dev(torch.zeros_like(phi), skew) for _ in range(3)]]
    tau = [_dev(torch.zeros_like(phi), skew)]
    psi, tau = mgic.lpt_displacements_and_source(H, [phi], scale=-1.0, out=out, tau=tau)
    for c in range(3):
        _close(psi[0][c], -_g4(phi, c, h))
    D = [[_g4(psi[0][i], j, h) for j in range(3)] for i in range(3)]
    t = sum(D[i][i] * D[j][j] - D[i][j] ** 2 for i in range(3) for j in range(i))
    _close(tau[0], t - t.mean())
    a = [[_dev(0.02 * h * x / x.abs().max(), skew) for x in psi[0]]]
    b = [[_dev(0.01 * h * torch.randn((n,) * 3, generator=g, dtype=torch.float64, device="cuda:0"), skew)
          for _ in range(3)]]
    for second in (None, b):
        L = [x if second is None else x + y for x, y in zip(a[0], b[0])]
        M = [[_g4(L[i], j, h) + (1.0 if i == j else 0.0) for j in range(3)] for i in range(3)]
        det = (M[0][0] * (M[1][1] * M[2][2] - M[1][2] * M[2][1]) - M[0][1] * (M[1][0] * M[2][2] - M[1][2] * M[2][0])
               + M[0][2] * (M[1][0] * M[2][1] - M[1][1] * M[2][0]))
        want = 1.0 / det - 1.0
        delta = mgic.lpt_lla_density(H, a, second, delta=[_dev(torch.zeros_like(phi), skew)])
        err = float((delta[0] - (want - want.mean())).abs().max())
        assert err <= TOL * max(1.0, float(want.abs().max())), err
