"""The work that a program using this library has it do, one case per path and size.

`listed()` holds the cases, `draw()` gives further ones over the same ranges, `prepare()` makes the
inputs and the workspaces a program keeps, `run()` is one pass through the public entry points,
`work()` its compulsory bytes and operations and `exact()` the same outputs in plain 64-bit torch.
"""

import math

import torch

from paper_1103_6031_amd import inputs, mgic

BOX = inputs.BOX
TOL = 1e-10
DEV = "cuda:0"


# ------------------------------------------------------------------------------------------------
# cases
# ------------------------------------------------------------------------------------------------

def listed():
    return [
        # the smallest production call: one 64^3 box in FP64, first order; launches and latency
        dict(name="1lpt 64 fp64", kind="lpt", n=64, prec="fp64", order=1, grad=4),
        # a size that is no power of two (3 * 2^5), second order, mixed precision
        dict(name="2lpt 96 mixed", kind="lpt", n=96, prec="mixed", order=2, grad=4),
        # the ordinary unigrid run and the library's headline: 256^3, second order, mixed
        dict(name="2lpt 256 mixed", kind="lpt", n=256, prec="mixed", order=2, grad=4),
        # the largest: a 512^3 box in FP64, first order; its arrays are far beyond every cache
        dict(name="1lpt 512 fp64", kind="lpt", n=512, prec="fp64", order=1, grad=4),
        # the zoom-in run: 128^3 base and three nested 128^3 patches, second order, mixed
        dict(name="zoom 128+3x128 mixed", kind="zoom", n=128, patches="128,128,128", prec="mixed", order=2, lap=2),
        # the same hierarchy with the sixth-order operators, FP64 only
        dict(name="zoom 128+3x128 order 6", kind="zoom", n=128, patches="128,128,128", prec="fp64", order=2, lap=6),
        # an ensemble of small boxes of mixed sizes in one call
        dict(name="batch 64 mixed", kind="batch", count=64, pick=1, prec="mixed"),
        # one 256^3 solve with the fourth-order Laplacian
        dict(name="level 256 order 4", kind="ho", n=256, lap=4, prec="fp64"),
        # the k-space correction of a unigrid run's displacements
        dict(name="hybrid 256 periodic", kind="hybrid", nx=256, ny=256, nz=256, isolated=False, lap=2, grad=4),
        # the same on the finest patch of a zoom run: isolated, ragged
        dict(name="hybrid 96x112x120 isolated", kind="hybrid", nx=96, ny=112, nz=120, isolated=True, lap=2, grad=4),
        # the density of a zoom run from white noise: the source of its solve
        dict(name="density 128+3x128", kind="density", n=128, patches="128,128,128", subgrid=True),
        # the baryon density of a unigrid second-order run
        dict(name="lla 256", kind="lla", n=256, sets=2),
    ]


def draw(rng):
    """One more case: sizes from 16^3 (the smallest boxes of the tests) to those listed."""
    kind = rng.choice(["lpt", "lpt", "lpt", "zoom", "zoom", "batch", "ho", "hybrid", "deconv", "density", "lla"])
    if kind == "lpt":
        n = rng.choice([16, 20, 24, 28, 32, 40, 48, 56, 64, 80, 96, 112, 128, 160, 192, 224, 256, 320, 384])
        return dict(kind=kind, n=n, prec=rng.choice(["fp64", "mixed"]), order=1 if n > 256 else rng.choice([1, 2]),
                    grad=rng.choice([4, 4, 6]))
    if kind == "zoom":                       # the serving range: bases of 64-256, patches of 64-128
        n, patches = rng.choice([64, 128, 256]), []
        for _ in range(rng.choice([1, 2, 3])):
            patches.append(rng.choice([m for m in (64, 80, 96, 112, 128) if m <= min([n] + patches)]))
        lap = rng.choice([2, 2, 2, 4, 6])
        return dict(kind=kind, n=n, patches=",".join(map(str, patches)), order=rng.choice([1, 2]), lap=lap,
                    prec="fp64" if lap > 2 else rng.choice(["fp64", "mixed"]))
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(6, 64), pick=rng.randint(2, 10 ** 6),
                    prec=rng.choice(["fp64", "mixed"]))
    if kind == "ho":
        return dict(kind=kind, n=rng.choice([32, 64, 128, 256]), lap=rng.choice([4, 6]),
                    prec=rng.choice(["fp64", "mixed"]))
    if kind in ("hybrid", "deconv"):
        iso = rng.random() < 0.5
        side = [rng.randint(20, 160) if iso else rng.choice([32, 64, 128, 256]) for _ in range(3)]
        c = dict(kind=kind, nx=side[0], ny=side[1], nz=side[2], isolated=iso)
        if kind == "hybrid":
            return dict(c, lap=rng.choice([2, 4, 6]), grad=rng.choice([4, 6]))
        return dict(c, window=rng.choice(["fv", "sg"]))
    if kind == "density":
        n, patches = rng.choice([64, 128]), []
        for _ in range(rng.choice([1, 2, 3])):
            patches.append(rng.choice([m for m in (16, 32, 64, 128) if m <= min([n] + patches)]))
        return dict(kind=kind, n=n, patches=",".join(map(str, patches)), subgrid=rng.random() < 0.5)
    return dict(kind=kind, n=rng.choice([32, 48, 64, 80, 96, 112, 128, 160, 192, 224, 256]), sets=rng.choice([1, 2]))


def _layout(c):
    """The case's nested patches, each centred in its parent: [(n3, off3), ...]."""
    out, parent = [], c["n"]
    for m in (int(v) for v in c["patches"].split(",")):
        out.append(((m,) * 3, ((parent - m // 2) // 2,) * 3))
        parent = m
    return out


def _batch_sizes(c):
    """Sizes of an ensemble: the library's own 64 instances (pick = 1), else a choice of its sizes."""
    if c["pick"] == 1:
        return [n for n, _, _ in inputs.c4_instances(c["count"])]
    g = torch.Generator().manual_seed(c["pick"])
    return [[32, 48, 64, 96, 128][i] for i in torch.randint(0, 5, (c["count"],), generator=g).tolist()]


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFF)


def _modes(shape, h):
    """Angular wave numbers of an rfftn of this shape, each with the axes it does not vary over as 1."""
    out = []
    for a, n in enumerate(shape):
        k = (torch.fft.rfftfreq if a == 2 else torch.fft.fftfreq)(n, d=h, dtype=torch.float64, device=DEV)
        out.append((2.0 * math.pi * k).reshape([-1 if b == a else 1 for b in range(3)]))
    return out


def _bbks(k, gamma=inputs.GAMMA):
    q = torch.where(k > 0, k, torch.ones_like(k)) / gamma
    t = torch.log1p(2.34 * q) / (2.34 * q) * (1.0 + 3.89 * q + (16.1 * q) ** 2 + (5.46 * q) ** 3
                                              + (6.71 * q) ** 4) ** -0.25
    return torch.where(k > 0, k * t * t, torch.zeros_like(k))


def _coloured(shape, h, g, slope=None, above=None):
    """White noise times sqrt(P(k) / h^3): BBKS, or k^slope; only modes above a wave number if given."""
    mu = torch.randn(shape, generator=g, dtype=torch.float64, device=DEV)
    kx, ky, kz = _modes(shape, h)
    k = torch.sqrt(kx * kx + ky * ky + kz * kz)
    if slope is None:
        P = _bbks(k)
    else:
        P = torch.where(k > 0, torch.where(k > 0, k, torch.ones_like(k)) ** slope, torch.zeros_like(k))
    amp = torch.sqrt(P / h ** 3)
    if above is not None:
        amp = amp * (torch.maximum(torch.maximum(kx.abs(), ky.abs()), kz.abs()) > above)
    return torch.fft.irfftn(torch.fft.rfftn(mu) * amp, s=shape).contiguous()


def _density(n, g, slope=None):
    """A periodic density of the library's rms, and the factor that gave it that rms."""
    d = _coloured((n,) * 3, BOX / n, g, slope)
    alpha = float(inputs.DELTA_RMS / torch.sqrt((d * d).mean()))
    return d * alpha, alpha


def _means8(x):
    a, b, c = x.shape
    return x.reshape(a // 2, 2, b // 2, 2, c // 2, 2).mean(dim=(1, 3, 5))


def _repeat8(x):
    return x.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)


def _children(parent, off, n):
    """Conservative tri-cubic interpolation of the parent cells under a patch."""
    w = (inputs._CUBIC_W).tolist()
    c = parent
    for a in range(3):
        i = torch.arange(off[a], off[a] + n[a] // 2, device=DEV)
        at = [torch.index_select(c, a, (i + s) % parent.shape[a]) for s in (-2, -1, 0, 1, 2)]
        lo = w[0] * at[3] + w[1] * at[2] + w[2] * at[1] + w[3] * at[0]
        hi = w[0] * at[1] + w[1] * at[2] + w[2] * at[3] + w[3] * at[4]
        shape = list(lo.shape)
        shape[a] *= 2
        c = torch.stack((lo, hi), dim=a + 1).reshape(shape)
    own = parent[tuple(slice(off[a], off[a] + n[a] // 2) for a in range(3))]
    return c + _repeat8(own - _means8(c))


def _nested(n, patches, g):
    """Density on a base and its patches: each the parent interpolated, plus power of its own."""
    base, alpha = _density(n, g)
    out, h = [base], BOX / n
    for m, off in patches:
        s = alpha * _coloured(m, h / 2, g, above=math.pi / h)
        out.append((_children(out[-1], off, m) + s - _repeat8(_means8(s))).contiguous())
        h /= 2
    return out


def _displacement_field(n, seed, rms):
    """k-space displacements of a BBKS density: [x, y, z], as a first- or second-order set."""
    d, _ = _density(n, _gen(seed))
    k = _modes(d.shape, BOX / n)
    kk = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    kk[0, 0, 0] = 1.0
    t = torch.fft.rfftn(d) * (rms / inputs.DELTA_RMS) / kk
    return [torch.fft.irfftn(1j * kc * t, s=d.shape).contiguous() for kc in k]


def _work_space(nbytes):
    return mgic.Workspace(nbytes)


def prepare(case, seed):
    c, g = case, _gen(seed)
    s = dict(case=c)
    if c["kind"] == "lpt":
        n = c["n"]
        H = mgic.Hier(n, BOX / n)
        s["f"], _ = _density(n, g)
        s["o"] = mgic.make_opts(tol=TOL, prec=c["prec"], max_cycles=60)
        s.update(H=H, ws=_work_space(mgic.mg_workspace_bytes(H, s["o"])),
                 wl=_work_space(mgic.lpt_workspace_bytes(H, 2 if c["order"] == 2 else 1)))
    elif c["kind"] == "zoom":
        patches = _layout(c)
        H = mgic.Hier(c["n"], BOX / c["n"], patches)
        s["f"] = _nested(c["n"], patches, g)
        s["o"] = mgic.make_opts(tol=TOL, prec=c["prec"], max_cycles=60)
        need = mgic.mg_workspace_bytes(H, s["o"]) if c["lap"] == 2 else mgic.mg_ho_hierarchy_workspace_bytes(H, c["lap"])
        s.update(H=H, ws=_work_space(need), wl=_work_space(mgic.lpt_workspace_bytes(H, 2 if c["order"] == 2 else 1)))
    elif c["kind"] == "batch":
        sizes = _batch_sizes(c)
        slopes = (torch.rand(len(sizes), generator=torch.Generator().manual_seed(int(seed))) - 2.5).tolist()
        s["f"] = [_density(n, g, a)[0] for n, a in zip(sizes, slopes)]
        s["h"] = [BOX / n for n in sizes]
        s["o"] = mgic.make_opts(tol=TOL, prec=c["prec"], max_cycles=60)
        s["ws"] = _work_space(mgic.mg_batch_workspace_bytes(sizes, s["o"]))
    elif c["kind"] == "ho":
        s["f"], _ = _density(c["n"], g)
        s["o"] = mgic.make_opts(tol=TOL, prec=c["prec"], max_cycles=60)
        s["ws"] = _work_space(mgic.mg_ho_workspace_bytes(c["n"], c["lap"]))
    elif c["kind"] in ("hybrid", "deconv"):
        shape = (c["nx"], c["ny"], c["nz"])
        d = _coloured(shape, 1.0, g)
        s["f"] = d * (inputs.DELTA_RMS / torch.sqrt((d * d).mean()))
        s["ws"] = _work_space(mgic.spec_workspace_bytes(shape, c["isolated"]))
        if c["kind"] == "hybrid":            # the displacements that the correction is added to
            s["psi"] = [torch.randn(shape, generator=g, dtype=torch.float64, device=DEV) for _ in range(3)]
    elif c["kind"] == "density":
        patches = _layout(c)
        _, alpha = _density(c["n"], g)
        H = mgic.Hier(c["n"], BOX / c["n"], patches)
        table, s["dr"] = inputs.radial_transfer_table(alpha, H.h(H.nlev - 1))
        s["radial"] = torch.from_numpy(table).to(DEV)
        s["xi"] = [torch.randn(tuple(2 * v for v in H.dims(p)) if p else H.dims(0), generator=g,
                               dtype=torch.float64, device=DEV) for p in range(H.nlev)]
        s.update(H=H, ws=_work_space(mgic.ic_density_workspace_bytes(H)))
    else:
        s["H"] = mgic.Hier(c["n"], BOX / c["n"])
        s["disp"] = [_displacement_field(c["n"], seed + 1000 * i, r) for i, r in enumerate((0.1, 0.01)[:c["sets"]])]
        s["ws"] = _work_space(mgic.lpt_workspace_bytes(s["H"], 3))
    return s


# ------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------

def run(s):
    c = s["case"]
    if c["kind"] == "lpt":
        H, h = s["H"], BOX / c["n"]
        phi, _ = mgic.mg_solve_level(s["f"], h, opts=s["o"], workspace=s["ws"])
        if c["order"] == 1:
            return phi, mgic.lpt_displacements(H, [phi], scale=-1.0, workspace=s["wl"], grad_order=c["grad"])[0]
        psi, tau = mgic.lpt_displacements_and_source(H, [phi], scale=-1.0, workspace=s["wl"], grad_order=c["grad"])
        phi2, _ = mgic.mg_solve_level(tau[0], h, opts=s["o"], workspace=s["ws"])
        psi2 = mgic.lpt_displacements(H, [phi2], scale=-3.0 / 7.0, workspace=s["wl"], grad_order=c["grad"])
        return phi, psi[0], tau[0], phi2, psi2[0]
    if c["kind"] == "zoom":
        H, grad = s["H"], 6 if c["lap"] == 6 else 4

        def solve(f):
            if c["lap"] == 2:
                return mgic.mg_solve_hierarchy(H, f, opts=s["o"], workspace=s["ws"])[0]
            return mgic.mg_solve_hierarchy_ho(H, c["lap"], f, opts=s["o"], workspace=s["ws"])[0]

        phi = solve(s["f"])
        if c["order"] == 1:
            return phi, mgic.lpt_displacements(H, phi, scale=-1.0, workspace=s["wl"], grad_order=grad)
        psi, tau = mgic.lpt_displacements_and_source(H, phi, scale=-1.0, workspace=s["wl"], grad_order=grad)
        phi2 = solve(tau)
        return phi, psi, tau, phi2, mgic.lpt_displacements(H, phi2, scale=-3.0 / 7.0, workspace=s["wl"],
                                                           grad_order=grad)
    if c["kind"] == "batch":
        return mgic.mg_solve_batch(s["f"], s["h"], opts=s["o"], workspace=s["ws"])[0]
    if c["kind"] == "ho":
        return mgic.mg_solve_level_ho(s["f"], BOX / c["n"], c["lap"], opts=s["o"], workspace=s["ws"])[0]
    if c["kind"] == "hybrid":
        out = [p.clone() for p in s["psi"]]  # the call adds to its outputs; a program keeps its own
        return mgic.lpt_hybrid_correction(s["f"], 1.0, out, isolated=c["isolated"], lap_order=c["lap"],
                                          grad_order=c["grad"], scale=-1.0, workspace=s["ws"])
    if c["kind"] == "deconv":
        kind = mgic.SPEC_FV_DECONV if c["window"] == "fv" else mgic.SPEC_SG_DECONV
        return mgic.spec_deconvolve(s["f"], kind, isolated=c["isolated"], workspace=s["ws"])
    if c["kind"] == "density":
        return mgic.ic_multiscale_density(s["H"], s["radial"], s["dr"], s["xi"], subgrid=c["subgrid"],
                                          workspace=s["ws"])
    return mgic.lpt_lla_density(s["H"], [s["disp"][0]], [s["disp"][1]] if c["sets"] == 2 else None,
                                workspace=s["ws"])


# ------------------------------------------------------------------------------------------------
# compulsory work
# ------------------------------------------------------------------------------------------------

# Ten V(2,2) cycles of 8 half-sweeps (2 flops per stencil point and updated cell), on a grid and its
# coarsenings (8/7 of its cells).
def _solve_flops(cells, lap):
    return 10 * 4 * cells * 8 / 7 * 2 * (3 * lap + 1)


def work(case):
    c = case
    if c["kind"] == "lpt":
        cells = c["n"] ** 3
        words = 1 + 4 if c["order"] == 1 else 1 + 9
        return dict(bytes=8 * words * cells, flops=c["order"] * (_solve_flops(cells, 2) + 3 * 8 * cells))
    if c["kind"] == "zoom":
        cells = c["n"] ** 3 + sum(int(m) ** 3 for m in c["patches"].split(","))
        words = 1 + 4 if c["order"] == 1 else 1 + 9
        return dict(bytes=8 * words * cells, flops=c["order"] * (_solve_flops(cells, c["lap"]) + 3 * 8 * cells))
    if c["kind"] == "batch":
        cells = sum(n ** 3 for n in _batch_sizes(c))
        return dict(bytes=16 * cells, flops=_solve_flops(cells, 2))
    if c["kind"] == "ho":
        return dict(bytes=16 * c["n"] ** 3, flops=_solve_flops(c["n"] ** 3, c["lap"]))
    if c["kind"] in ("hybrid", "deconv"):
        cells = c["nx"] * c["ny"] * c["nz"]
        grid = [1 << (2 * n - 1).bit_length() for n in (c["nx"], c["ny"], c["nz"])] if c["isolated"] else [
            c["nx"], c["ny"], c["nz"]]
        points = math.prod(grid)
        transforms = 4 if c["kind"] == "hybrid" else 2          # of real data: half of 5 N log2 N
        return dict(bytes=8 * cells * (1 + 6 if c["kind"] == "hybrid" else 2),
                    flops=transforms * 2.5 * points * math.log2(points))
    if c["kind"] == "density":
        dims = [c["n"]] + [int(m) for m in c["patches"].split(",")]
        out = sum(m ** 3 for m in dims)
        noise = dims[0] ** 3 + sum((2 * m) ** 3 for m in dims[1:])
        # per level a kernel, its noise and its density transformed; per patch the noise refined
        # (two transforms) and the coarse contribution convolved
        flops = sum(2.5 * (2 * m if p else m) ** 3 * 3 * math.log2(2 * m) * (3 if p == 0 else 7)
                    for p, m in enumerate(dims))
        return dict(bytes=8 * (out + noise), flops=flops)
    cells = c["n"] ** 3
    return dict(bytes=8 * cells * (3 * c["sets"] + 1), flops=cells * (9 * 8 + 20))


# ------------------------------------------------------------------------------------------------
# the same in plain 64-bit torch
# ------------------------------------------------------------------------------------------------

_LAP = {2: ((1, 2.0), (0, -2.0)), 4: ((2, -1 / 6), (1, 16 / 6), (0, -2.5)),
        6: ((3, 1 / 45), (2, -0.3), (1, 3.0), (0, -49 / 18))}     # symbol: sum of a_j cos(j k), j = 0 once
_GRAD = {4: ((1, 8 / 12), (2, -1 / 12)), 6: ((1, 45 / 60), (2, -9 / 60), (3, 1 / 60))}


def _laplacian_symbol(shape, lap):
    k = _modes(shape, 1.0)
    return sum(sum(a * torch.cos(j * kc) for j, a in _LAP[lap]) for kc in k)


def _poisson(f, h, lap):
    lam = _laplacian_symbol(f.shape, lap)
    lam[0, 0, 0] = 1.0
    t = torch.fft.rfftn(f) / lam * (h * h)
    t[0, 0, 0] = 0.0
    return torch.fft.irfftn(t, s=f.shape)


def _diff(x, axis, h, grad):
    return sum(a * (torch.roll(x, -j, axis) - torch.roll(x, j, axis)) for j, a in _GRAD[grad]) / h


def _tau(phi, h, grad):
    g = [_diff(phi, a, h, grad) for a in range(3)]
    t = torch.zeros_like(phi)
    for i in range(3):
        for j in range(i):
            t += _diff(g[i], i, h, grad) * _diff(g[j], j, h, grad) - _diff(g[j], i, h, grad) ** 2
    return t - t.mean()


def exact(case, seed):
    c = case
    if c["kind"] in ("zoom", "density"):
        return None                          # composite systems: no direct solution in plain torch
    s = prepare(case, seed)
    if c["kind"] == "lpt":
        h = BOX / c["n"]
        phi = _poisson(s["f"], h, 2)
        psi = [-_diff(phi, a, h, c["grad"]) for a in range(3)]
        if c["order"] == 1:
            return phi, psi
        tau = _tau(phi, h, c["grad"])
        phi2 = _poisson(tau, h, 2)
        return phi, psi, tau, phi2, [-3.0 / 7.0 * _diff(phi2, a, h, c["grad"]) for a in range(3)]
    if c["kind"] == "batch":
        return [_poisson(f, h, 2) for f, h in zip(s["f"], s["h"])]
    if c["kind"] == "ho":
        return _poisson(s["f"], BOX / c["n"], c["lap"])
    if c["kind"] in ("hybrid", "deconv"):
        shape = tuple(s["f"].shape)
        grid = tuple(1 << (2 * n - 1).bit_length() for n in shape) if c["isolated"] else shape
        own = tuple(slice(0, n) for n in shape)
        k = _modes(grid, 1.0)
        t = torch.fft.rfftn(s["f"], s=grid)
        if c["kind"] == "deconv":
            for kc in k:
                t = t / (torch.sinc(kc / (2 * math.pi)) if c["window"] == "fv" else torch.cos(kc / 4))
            return torch.fft.irfftn(t, s=grid)[own]
        lam = _laplacian_symbol(grid, c["lap"])
        kk = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
        lam[0, 0, 0] = kk[0, 0, 0] = 1.0
        out = []
        for a in range(3):
            sym = -k[a] / kk - 2.0 * sum(b * torch.sin(j * k[a]) for j, b in _GRAD[c["grad"]]) / lam
            sym[0, 0, 0] = 0.0
            sym.narrow(a, grid[a] // 2, 1).zero_()          # the Nyquist plane gets no correction
            out.append(s["psi"][a] + torch.fft.irfftn(-1j * sym * t, s=grid)[own])
        return out
    L = [sum(d[a] for d in s["disp"]) for a in range(3)]
    h = BOX / c["n"]
    J = [[_diff(L[i], j, h, 4) + (1.0 if i == j else 0.0) for j in range(3)] for i in range(3)]
    det = (J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) - J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0])
           + J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]))
    d = 1.0 / det - 1.0
    return [d - d.mean()]
