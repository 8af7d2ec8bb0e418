"""The higher-order kernels that do several steps in one launch against the one-step kernels, launch by launch: the
same operations on every value in the same order, so the same bits.

k_ho_sweep against two half-sweeps; k_ho_tail against the V-cycle of its levels step by step; the marched half-sweep
of a large patch against the row kernel on its two halves, whose ghost layers at the cut are the patch's own cells.
The launchers are the library's internal ones, called by their linker names.
"""

import ctypes

import numpy as np
import pytest

from gpu_util import needs_gpu, note

pytestmark = [pytest.mark.gpu, needs_gpu]

_S = "P12ihipStream_t"
NAMES = {"half": "_ZN4mgic14launch_ho_halfI%sEEvPKT_PS1_S3_idii" + _S + "P11ihipEvent_tS8_",
         "sweep": "_ZN4mgic15launch_ho_sweepI%sEEvPKT_PS1_S3_idi" + _S + "P11ihipEvent_tS8_",
         "tail": "_ZN4mgic14launch_ho_tailI%sEE10hipError_tPT_PKS2_idiiib" + _S,
         "restrict": "_ZN4mgic24launch_ho_resid_restrictI%sEEvPKT_S3_PS1_S4_S4_idi" + _S,
         "fas": "_ZN4mgic13launch_ho_fasI%sEEvPKT_PS1_idi" + _S,
         "prolong": "_ZN4mgic17launch_ho_prolongI%sEEvPT_PKS1_S4_i" + _S}
P, I, D = ctypes.c_void_p, ctypes.c_int, ctypes.c_double
ARGS = {"half": [P, P, P, I, D, I, I, P, P, P], "sweep": [P, P, P, I, D, I, P, P, P],
        "tail": [P, P, I, D, I, I, I, ctypes.c_bool, P], "restrict": [P, P, P, P, P, I, D, I, P],
        "fas": [P, P, I, D, I, P], "prolong": [P, P, P, I, P]}


def _fn(name, double):
    from paper_1103_6031_amd import mgic
    fn = getattr(mgic._lib, NAMES[name] % ("d" if double else "f"))
    fn.argtypes, fn.restype = ARGS[name], I if name == "tail" else None
    return lambda *a: fn(*[x.data_ptr() if hasattr(x, "data_ptr") else x for x in a])


def _st():
    from paper_1103_6031_amd import mgic
    return mgic._stream()


def _field(n, seed, double):
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    t = torch.randn((n,) * 3, generator=g, dtype=torch.float64, device="cuda:0")
    return t if double else t.float()


@pytest.mark.parametrize("double", [True, False])
@pytest.mark.parametrize("order,lg", [(2, 5), (2, 6), (2, 8), (4, 5), (4, 6), (4, 8), (6, 7), (6, 8)])
def test_sweep_is_two_half_sweeps(order, lg, double):
    import torch
    half, sweep = _fn("half", double), _fn("sweep", double)
    u, f = _field(1 << lg, lg, double), _field(1 << lg, 50 + lg, double)
    tmp, want, got = (torch.empty_like(u) for _ in range(3))
    note("ho bits: sweep order %d 2^%d double=%s" % (order, lg, double))
    half(u, tmp, f, lg, 0.37, order, 0, _st(), None, None)
    half(tmp, want, f, lg, 0.37, order, 1, _st(), None, None)
    sweep(u, got, f, lg, 0.37, order, _st(), None, None)
    torch.cuda.synchronize()
    assert torch.equal(got, want)


@pytest.mark.parametrize("double", [True, False])
@pytest.mark.parametrize("fas", [False, True])
@pytest.mark.parametrize("order,lg,nu", [(2, 4, (2, 2)), (4, 4, (2, 2)), (4, 4, (1, 3)), (6, 4, (2, 2)), (6, 3, (2, 1)),
                                         (4, 1, (2, 2)), (2, 2, (0, 2))])
def test_tail_is_its_steps(order, lg, nu, fas, double):
    import torch
    half, restrict = _fn("half", double), _fn("restrict", double)
    add, prolong, tail = _fn("fas", double), _fn("prolong", double), _fn("tail", double)
    h = 0.21
    u = [_field(1 << lg, lg, double)] + [torch.empty((1 << k,) * 3, dtype=torch.float64 if double else torch.float32,
                                                     device="cuda:0") for k in range(lg - 1, -1, -1)]
    f = [_field(1 << lg, 60 + lg, double)] + [torch.empty_like(x) for x in u[1:]]
    old, tmp = [torch.empty_like(x) for x in u], [torch.empty_like(x) for x in u]
    got, rhs = u[0].clone(), f[0].clone()

    def smooth(k, sweeps):
        for _ in range(sweeps):
            half(u[k], tmp[k], f[k], lg - k, h * 2 ** k, order, 0, _st(), None, None)
            half(tmp[k], u[k], f[k], lg - k, h * 2 ** k, order, 1, _st(), None, None)

    note("ho bits: tail order %d 2^%d nu=%s fas=%s double=%s" % (order, lg, nu, fas, double))
    if fas:
        add(u[0], f[0], lg, h, order, _st())
    for k in range(lg):
        smooth(k, nu[0])
        restrict(u[k], f[k], u[k + 1], old[k + 1], f[k + 1], lg - k - 1, h * 2 ** k, order, _st())
        if k + 1 < lg:
            add(u[k + 1], f[k + 1], lg - k - 1, h * 2 ** (k + 1), order, _st())
    u[lg].zero_()
    for k in range(lg - 1, -1, -1):
        prolong(u[k], u[k + 1], old[k + 1], lg - k, _st())
        smooth(k, nu[1])
    assert tail(got, rhs, lg, h, order, nu[0], nu[1], fas, _st()) == 0
    torch.cuda.synchronize()
    assert torch.equal(got, u[0])


class Patch(ctypes.Structure):
    _fields_ = [("n", I * 3), ("off", I * 3), ("pn", I * 3), ("pper", I), ("h", D)]


@pytest.mark.parametrize("order,n", [(4, (132, 130, 138)), (6, (130, 132, 134)), (2, (164, 162, 166))])
def test_marched_half_sweep_is_the_row_kernels(order, n):
    import torch
    from paper_1103_6031_amd import mgic
    fn = mgic._lib._ZN4mgic15launch_hoz_halfEPKdPdS1_S1_RKNS_8HozPatchEiiP12ihipStream_t
    fn.argtypes, fn.restype = [P, P, P, P, ctypes.POINTER(Patch), I, I, P], None
    R = order // 2
    rng = torch.Generator(device="cuda:0").manual_seed(order)

    def rand(*shape):
        return torch.randn(shape, generator=rng, dtype=torch.float64, device="cuda:0")

    u, f = rand(*n), rand(*n)
    x, y, z = ([rand(R, *s) for _ in range(2)] for s in ((n[1], n[2]), (n[0], n[2]), (n[0], n[1])))

    def run(u, f, ghosts, colour):
        P_ = Patch((I * 3)(*u.shape), (I * 3)(), (I * 3)(*u.shape), 0, 0.43)
        g = torch.cat([t.reshape(-1) for t in ghosts]).contiguous()
        out = torch.full_like(u, float("nan"))
        fn(u.data_ptr(), out.data_ptr(), f.data_ptr(), g.data_ptr(), ctypes.byref(P_), order, colour, _st())
        torch.cuda.synchronize()
        return out

    cut = n[0] // 4 * 2                       # an even plane: the halves' colours are the patch's
    line = 1 << (21 if R > 1 else 22)         # cells from which a patch is marched
    assert max(cut, n[0] - cut) * n[1] * n[2] < line <= n[0] * n[1] * n[2]
    for colour in (0, 1):
        note("ho bits: marched half-sweep order %d colour %d" % (order, colour))
        whole = run(u, f, x + y + z, colour)
        low = run(u[:cut].contiguous(), f[:cut].contiguous(),
                  [x[0], u[cut:cut + R]] + [t[:, :cut].contiguous() for t in y + z], colour)
        high = run(u[cut:].contiguous(), f[cut:].contiguous(),
                   [u[cut - R:cut].flip(0), x[1]] + [t[:, cut:].contiguous() for t in y + z], colour)
        assert torch.equal(whole[:cut], low) and torch.equal(whole[cut:], high)
