"""Every transform length on every axis of the real-field FFT, against the oracle.

Each length 2 .. 1024 has its own stages, tile shape and thread mapping, as strided lines (x, y) and as
contiguous real lines (z); odd isolated extents and arrays that are not 16-byte aligned take the
point-by-point accesses of the z passes.  Tolerance: numpy's FFT and this one are both backward
stable, error ~ eps log2(P) of the transform's norm: 1e-12 of the largest magnitude is a few hundred
eps, as for the other spectral tests.
"""

import numpy as np
import pytest

from gpu_util import needs_gpu, note, to_host

pytestmark = [pytest.mark.gpu, needs_gpu]

TOL = 1e-12


def _dev(a, skew):
    """A device copy of a, starting `skew` doubles into its allocation."""
    import torch
    buf = torch.empty(a.size + skew, dtype=torch.float64, device="cuda:0")
    t = buf[skew:].view(a.shape)
    t.copy_(torch.from_numpy(a))
    return t


def _close(got, want):
    scale = max(float(np.max(np.abs(want))), 1e-300)
    err = float(np.max(np.abs(got - want)))
    assert err <= TOL * scale, (err, scale)


@pytest.mark.parametrize("skew", [0, 1])
@pytest.mark.parametrize("lg", range(1, 11))
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_deconvolution_of_every_length(axis, lg, skew):
    from oracle import spectral
    from paper_1103_6031_amd import mgic
    shape = [4, 2, 8]
    shape[axis] = 1 << lg
    f = np.random.default_rng(100 * axis + lg).standard_normal(shape)
    note("spectral lengths: shape %s skew %d" % (shape, skew))
    out = _dev(np.zeros(shape), skew)
    mgic.spec_deconvolve(_dev(f, skew), mgic.SPEC_FV_DECONV, out=out)
    _close(to_host(out), spectral.fv_deconvolve(f))


@pytest.mark.parametrize("shape", [(3, 5, 301), (3, 301, 5), (301, 5, 3), (17, 33, 66), (1, 1, 1)])
@pytest.mark.parametrize("skew", [0, 1])
def test_isolated_hybrid_of_odd_extents(shape, skew):
    from oracle import spectral
    from paper_1103_6031_amd import mgic
    rng = np.random.default_rng(sum(shape))
    f, base = rng.standard_normal(shape), rng.standard_normal((3,) + shape)
    note("spectral lengths: isolated hybrid %s skew %d" % (shape, skew))
    out = [_dev(base[c], skew) for c in range(3)]
    mgic.lpt_hybrid_correction(_dev(f, skew), 0.37, out, isolated=True, lap_order=4, grad_order=6, scale=-1.3)
    corr = spectral.hybrid_correction(f, 0.37, 4, 6, -1.3, periodic=False)
    for c in range(3):
        got = to_host(out[c]) - base[c]      # cancels to eps of the sum's largest term
        assert np.max(np.abs(got - corr[c])) <= TOL * max(np.max(np.abs(corr[c])), np.max(np.abs(base[c])))


def test_every_length_in_a_hybrid_x_pass():
    from oracle import spectral
    from paper_1103_6031_amd import mgic
    import torch
    for lg in range(1, 11):
        shape = (1 << lg, 4, 2)
        f = np.random.default_rng(lg).standard_normal(shape)
        note("spectral lengths: hybrid x length %d" % (1 << lg))
        out = [torch.zeros(shape, dtype=torch.float64, device="cuda:0") for _ in range(3)]
        mgic.lpt_hybrid_correction(_dev(f, 0), 0.5, out)
        corr = spectral.hybrid_correction(f, 0.5, 2, 4, 1.0)
        for c in range(3):
            _close(to_host(out[c]), corr[c])
