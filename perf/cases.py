"""The work that users of this library have it do, as a list of timed cases.

Every case is one pass through the public entry points of
paper_1412_0934_amd.godunov, in the library's default configuration, on
inputs that are on the GPU already:

    step      one patch or periodic box (PLM or PPM, optionally with the CFL
              reduction before it or fused into it)
    batch     many uneven ghost-zoned patches with their boundary fluxes
    adjoint   the reverse of one step
    rollout   a differentiable rollout: forward, then the gradient
    mhd       the ideal-MHD step
    amr       the two-level step: ghost fill, both levels, refluxing

Inputs are made on the GPU from a seed: log-normal turbulence, shocked
patches, shock tubes and smooth boxes as in paper_1412_0934_amd.inputs.
exact() evaluates the same schemes in plain torch, in float64, from their
definitions in include/godunov.h.
"""
import math

import numpy as np
import torch

from paper_1412_0934_amd import godunov

GAMMA = 5.0 / 3.0
FLOOR = 1e-10
CFL = 0.5
DTYPE = {"f64": torch.float64, "f32": torch.float32}


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # one small ghosted patch stepped by itself, as a code that does not
        # batch its refinement patches does thousands of times: launch latency
        dict(name="patch_8", kind="step", init="shock", nx=8, ny=8, nz=8, dtype="f64",
             limiter="minmod", riemann="hllc", cfl="given", bflux=True, reuse=True),
        # the shock-tube patch of the quick start: cfl_dt, then the step with
        # its boundary fluxes, outputs allocated by the call
        dict(name="patch_sod_32", kind="step", init="sod", nx=32, ny=32, nz=32, dtype="f64",
             limiter="minmod", riemann="hllc", cfl="before", bflux=True, reuse=False),
        # the main box: one time step of periodic turbulence, its CFL fused
        dict(name="box_256", kind="step", init="turbulence", nx=256, ny=256, nz=256, dtype="f64",
             limiter="minmod", riemann="hllc", cfl="fused", bflux=False, reuse=True),
        # a box whose extents no tile divides, in single precision, with the
        # sharper limiter
        dict(name="box_odd_f32", kind="step", init="turbulence", nx=250, ny=190, nz=141,
             dtype="f32", limiter="mc", riemann="hllc", cfl="fused", bflux=False, reuse=True),
        # PPM on the main box
        dict(name="box_ppm_256", kind="step", init="turbulence", nx=256, ny=256, nz=256,
             dtype="f64", limiter="ppm", riemann="hllc", cfl="fused", bflux=False, reuse=True),
        # one level of an AMR run: 4096 cubic patches of 8..32 cells
        dict(name="batch_4096", kind="batch", npatch=4096, sizes="8,16,24,32",
             probs="0.5,0.3,0.15,0.05", cubic=True, layout=5, ng=2, dtype="f64",
             limiter="minmod", riemann="hllc", cfl="fused"),
        # a coarser level in single precision: few patches, no two extents
        # alike, the more diffusive solver
        dict(name="batch_uneven_f32", kind="batch", npatch=500, sizes="6,11,16,21,27,40",
             probs="0.2,0.2,0.2,0.2,0.1,0.1", cubic=False, layout=6, ng=2, dtype="f32",
             limiter="mc", riemann="hll", cfl="given"),
        # PPM with characteristic tracing on a batch
        dict(name="batch_ppm_ct_1024", kind="batch", npatch=1024, sizes="8,16,24,32",
             probs="0.5,0.3,0.15,0.05", cubic=True, layout=7, ng=3, dtype="f64",
             limiter="ppm_ct", riemann="hllc", cfl="fused"),
        # reverse mode of one ghosted patch whose boundary fluxes carry
        # adjoints too
        dict(name="adjoint_patch", kind="adjoint", init="shock", nx=112, ny=84, nz=60,
             limiter="mc", riemann="hllc", periodic=False, bflux=True),
        # gradient of a rollout with respect to its initial state
        dict(name="rollout_128", kind="rollout", n=128, nsteps=10, every=5, limiter="minmod",
             riemann="hllc"),
        # ideal MHD, the next dt and cleaning speed from the same call
        dict(name="mhd_128", kind="mhd", nx=128, ny=128, nz=128, dtype="f64", limiter="minmod"),
        # one step of a two-level hierarchy
        dict(name="amr_128", kind="amr", nc=128, npatch=1024, most=12, layout=11, dtype="f64",
             limiter="minmod", riemann="hllc"),
    ]


def _between(rng, lo, hi):
    """A size in [lo, hi], spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "box", "box", "batch", "batch", "adjoint",
                       "rollout", "mhd", "amr"])
    dtype = rng.choice(["f64", "f64", "f32"])
    limiter = rng.choice(["minmod", "minmod", "mc", "unlimited"])
    riemann = rng.choice(["hllc", "hllc", "hll"])
    if kind == "step":
        nx, ny, nz = (_between(rng, 6, 120) for _ in range(3))
        return dict(kind="step", init=rng.choice(["shock", "sod"]), nx=nx, ny=ny, nz=nz,
                    dtype=dtype, limiter=rng.choice([limiter, "ppm", "ppm_ct"]), riemann=riemann,
                    cfl=rng.choice(["given", "before", "fused"]), bflux=rng.random() < 0.8,
                    reuse=rng.random() < 0.5)
    if kind == "box":
        nx, ny, nz = (_between(rng, 24, 256) for _ in range(3))
        return dict(kind="step", init="turbulence", nx=nx, ny=ny, nz=nz, dtype=dtype,
                    limiter=rng.choice([limiter, "ppm", "ppm_ct"]), riemann=riemann, cfl="fused",
                    bflux=False, reuse=True)
    if kind == "batch":
        ppm = rng.random() < 0.35
        cubic = rng.random() < 0.5
        sizes = sorted({_between(rng, 6, 40) for _ in range(4)})
        npatch = _between(rng, 16, 1000 if ppm or max(sizes) > 28 else 3000)
        return dict(kind="batch", npatch=npatch, sizes=",".join(map(str, sizes)),
                    probs=",".join(["%.4f" % (1.0 / len(sizes))] * len(sizes)), cubic=cubic,
                    layout=rng.randrange(1000), ng=3 if ppm else rng.choice([2, 2, 3]),
                    dtype=dtype, limiter=rng.choice(["ppm", "ppm_ct"]) if ppm else limiter,
                    riemann=riemann, cfl=rng.choice(["given", "fused"]))
    if kind == "adjoint":
        nx, ny, nz = (_between(rng, 12, 128) for _ in range(3))
        periodic = rng.random() < 0.5
        return dict(kind="adjoint", init="turbulence" if periodic else "shock", nx=nx, ny=ny, nz=nz,
                    limiter=limiter, riemann=riemann, periodic=periodic,
                    bflux=not periodic and rng.random() < 0.5)
    if kind == "rollout":
        return dict(kind="rollout", n=_between(rng, 24, 120), nsteps=rng.randrange(3, 11),
                    every=rng.choice([2, 3, 5]), limiter=limiter, riemann=riemann)
    if kind == "mhd":
        nx, ny, nz = (_between(rng, 16, 144) for _ in range(3))
        return dict(kind="mhd", nx=nx, ny=ny, nz=nz, dtype=dtype, limiter=limiter)
    return dict(kind="amr", nc=rng.randrange(40, 121), npatch=_between(rng, 20, 800),
                most=rng.randrange(5, 13), layout=rng.randrange(1000), dtype=dtype,
                limiter=limiter, riemann=riemann)


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 62))


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)


def _conserved(rho, vx, vy, vz, p, B=None):
    e = p / (GAMMA - 1.0) + 0.5 * rho * (vx * vx + vy * vy + vz * vz)
    if B is None:
        return torch.stack([rho, rho * vx, rho * vy, rho * vz, e])
    e = e + 0.5 * (B[0] * B[0] + B[1] * B[1] + B[2] * B[2])
    return torch.stack([rho, rho * vx, rho * vy, rho * vz, e, *B, torch.zeros_like(rho)])


def _random_field(g, nx, ny, nz):
    """A unit-variance Gaussian random field with power spectrum k^-11/3."""
    m = max(nx, ny, nz)
    kx = torch.fft.rfftfreq(nx, device="cuda", dtype=torch.float64) * m
    ky = torch.fft.fftfreq(ny, device="cuda", dtype=torch.float64) * m
    kz = torch.fft.fftfreq(nz, device="cuda", dtype=torch.float64) * m
    kk = kx[None, None, :] ** 2 + ky[None, :, None] ** 2 + kz[:, None, None] ** 2
    amp = torch.where(kk > 0, kk.clamp(min=1e-30) ** (-11.0 / 12.0), torch.zeros_like(kk))
    white = torch.randn((nz, ny, nx), generator=g, device="cuda", dtype=torch.float64)
    f = torch.fft.irfftn(torch.fft.rfftn(white) * amp, s=(nz, ny, nx))
    f = f - f.mean()
    return f / f.std()


def _turbulence(seed, nx, ny, nz, mach=2.0, beta=None):
    g = _gen(seed)
    rho = torch.exp(_random_field(g, nx, ny, nz) - 0.5)
    v = [_random_field(g, nx, ny, nz) for _ in range(3)]
    scale = mach * math.sqrt(0.6) / torch.sqrt((v[0] ** 2 + v[1] ** 2 + v[2] ** 2).mean())
    p = 0.6 * rho / GAMMA
    B = None
    if beta is not None:
        B = [_random_field(g, nx, ny, nz) for _ in range(3)]
        b2 = (B[0] ** 2 + B[1] ** 2 + B[2] ** 2).mean()
        B = [b * torch.sqrt(2.0 * p.mean() / beta / b2) for b in B]
    return _conserved(rho, *[c * scale for c in v], p, B).contiguous(), 1.0 / max(nx, ny, nz)


def _smooth(seed, n):
    """A periodic box of a few low Fourier modes at 5% amplitude."""
    g = _gen(seed)
    x = (torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) / n
    f = []
    for _ in range(5):
        s = torch.zeros((n, n, n), device="cuda", dtype=torch.float64)
        for _ in range(8):
            k = torch.randint(-4, 5, (3,), generator=g, device="cuda").double() + 0.0
            ph = _uniform(g, 0.0, 2 * math.pi, 1)
            s += torch.sin(2 * math.pi * (k[0] * x[None, None, :] + k[1] * x[None, :, None]
                                          + k[2] * x[:, None, None]) + ph)
        f.append(s / s.abs().max().clamp(min=1e-30))
    c = math.sqrt(GAMMA)
    return _conserved(1 + 0.05 * f[0], 0.05 * c * f[1], 0.05 * c * f[2], 0.05 * c * f[3],
                      1 + 0.05 * f[4]).contiguous(), 1.0 / n


def _sod(seed, nx, ny, nz, ng):
    """A shock tube along x with 1% density noise and zero-gradient ghosts."""
    g = _gen(seed)
    left = (torch.arange(nx, device="cuda") < nx // 2)[None, None, :].expand(nz, ny, nx)
    one = torch.ones((nz, ny, nx), device="cuda", dtype=torch.float64)
    rho = torch.where(left, one, 0.125 * one) * (1 + 0.01 * _uniform(g, -1, 1, nz, ny, nx))
    p = torch.where(left, one, 0.1 * one)
    u = _conserved(rho, 0 * one, 0 * one, 0 * one, p)
    return _extend(u, ng, "edge").contiguous(), 1.0 / max(nx, ny, nz)


def _shocked(seed, dims, ng, dx):
    """Ghosted patches of the given extents, each a smooth background (1 +- 0.2)
    cut by a planar Mach-3 shock of random orientation, in one flat buffer:
    patch after patch, each [5][nz+2ng][ny+2ng][nx+2ng]."""
    g = _gen(seed)
    P = len(dims)
    d = torch.as_tensor(dims, device="cuda")
    e = d + 2 * ng
    cells = e.prod(1)
    start = torch.cumsum(cells, 0) - cells
    pid = torch.repeat_interleave(torch.arange(P, device="cuda"), cells)
    loc = torch.arange(int(cells.sum()), device="cuda") - start[pid]
    ex, ey = e[pid, 0], e[pid, 1]
    idx = [loc % ex, (loc // ex) % ey, loc // (ex * ey)]
    origin = _uniform(g, 0, 1, P, 3)
    X = [origin[pid, a] + (idx[a] - ng + 0.5) * dx for a in range(3)]

    def wave():
        k = torch.randint(1, 3, (P, 3), generator=g, device="cuda").double()
        k = k * (2 * torch.randint(0, 2, (P, 3), generator=g, device="cuda") - 1)
        ph = _uniform(g, 0, 2 * math.pi, P)
        return torch.sin(2 * math.pi * sum(k[pid, a] * X[a] for a in range(3)) + ph[pid])

    def unit():
        v = torch.randn((P, 3), generator=g, device="cuda", dtype=torch.float64)
        return v / v.norm(dim=1, keepdim=True)

    rho, p, vm = 1 + 0.2 * wave(), 1 + 0.2 * wave(), 0.1 * wave()
    ev, nrm = unit(), unit()
    through = origin + dx * _uniform(g, 0, 1, P, 3) * d
    c = torch.sqrt(GAMMA * p / rho)
    m2 = 9.0
    ratio = (GAMMA + 1) * m2 / ((GAMMA - 1) * m2 + 2)
    pjump = (2 * GAMMA * m2 - (GAMMA - 1)) / (GAMMA + 1)
    du = (1 - 1 / ratio) * 3.0 * c
    behind = sum(nrm[pid, a] * (X[a] - through[pid, a]) for a in range(3)) <= 0
    v = [vm * ev[pid, a] + torch.where(behind, du * nrm[pid, a], torch.zeros_like(du))
         for a in range(3)]
    U = _conserved(torch.where(behind, rho * ratio, rho), *v, torch.where(behind, p * pjump, p))
    out = torch.empty(5 * U.shape[1], device="cuda", dtype=torch.float64)
    at = 5 * start[pid] + loc
    for q in range(5):
        out[at + q * cells[pid]] = U[q]
    return out


def _batch_dims(case):
    r = np.random.default_rng(case["layout"])
    sizes = [int(s) for s in case["sizes"].split(",")]
    probs = np.array([float(s) for s in case["probs"].split(",")])
    n = r.choice(sizes, size=(case["npatch"], 1 if case["cubic"] else 3), p=probs / probs.sum())
    return np.repeat(n, 3, axis=1) if case["cubic"] else n


def _offsets(dims, ng):
    def off(v):
        return np.concatenate([[0], np.cumsum(v)[:-1]]).astype(np.int64), int(v.sum())
    d = np.asarray(dims, dtype=np.int64)
    fl = 10 * (d[:, 2] * d[:, 1] + d[:, 2] * d[:, 0] + d[:, 1] * d[:, 0])
    return off(5 * np.prod(d + 2 * ng, axis=1)), off(5 * np.prod(d, axis=1)), off(fl)


def _hierarchy(case):
    """Disjoint random patches, (lo, n) in coarse cells, strictly inside the
    box; half of them placed against an existing one."""
    nc, most = case["nc"], case["most"]
    r = np.random.default_rng(case["layout"])
    taken = np.zeros((nc, nc, nc), dtype=bool)
    lo, size = [], []
    for _ in range(4 * case["npatch"]):
        if len(lo) == case["npatch"]:
            break
        s = r.integers(2, most + 1, size=3)
        a = r.integers(2, nc - 1 - s)
        if lo and r.uniform() < 0.5:
            q, ax = r.integers(len(lo)), r.integers(3)
            a = lo[q] + r.integers(-1, 2, size=3)
            a[ax] = lo[q][ax] + size[q][ax] if r.uniform() < 0.5 else lo[q][ax] - s[ax]
        if (a < 2).any() or (a + s > nc - 2).any():
            continue
        box = taken[a[0]:a[0] + s[0], a[1]:a[1] + s[1], a[2]:a[2] + s[2]]
        if box.any():
            continue
        box[...] = True
        lo.append(a)
        size.append(s)
    return np.array(lo), np.array(size)


def _hierarchy_state(seed, case):
    """The same smooth state at the coarse cell centres and, in a full fine
    grid, at the fine ones."""
    g = _gen(seed)
    nc = case["nc"]
    k = torch.randint(1, 3, (5, 3), generator=g, device="cuda").double()
    k = k * (2 * torch.randint(0, 2, (5, 3), generator=g, device="cuda") - 1)
    ph = _uniform(g, 0, 2 * math.pi, 5)

    def at(n):
        x = (torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) / n
        f = [torch.sin(2 * math.pi * (k[i, 0] * x[None, None, :] + k[i, 1] * x[None, :, None]
                                      + k[i, 2] * x[:, None, None]) + ph[i]) for i in range(5)]
        return _conserved(1 + 0.2 * f[0], 0.3 * f[1], 0.3 * f[2], 0.3 * f[3], 1 + 0.2 * f[4])

    return at(nc), at(2 * nc)


def _signal_dt(prims, dx, cfl=CFL):
    """dt of the summed CFL condition from a list of primitive states."""
    s = 0.0
    for W in prims:
        c = torch.sqrt(GAMMA * W[4] / W[0])
        s = max(s, float((W[1].abs() + W[2].abs() + W[3].abs() + 3 * c).max()))
    return cfl * dx / s


def _scalar(x):
    return torch.tensor([float(x)], dtype=torch.float64, device="cuda")


def _inputs(case, seed):
    """The arrays of a case (in its dtype) and its dt, as plain tensors."""
    dt = DTYPE[case.get("dtype", "f64")]
    kind = case["kind"]
    if kind in ("step", "adjoint"):
        n = (case["nx"], case["ny"], case["nz"])
        ng = 0 if case["init"] == "turbulence" else (3 if case["limiter"].startswith("ppm") else 2)
        if case["init"] == "turbulence":
            u, dx = _turbulence(seed, *n)
        elif case["init"] == "sod":
            u, dx = _sod(seed, *n, ng)
        else:
            dx = 1.0 / 256
            u = _shocked(seed, [n], ng, dx).view(5, n[2] + 2 * ng, n[1] + 2 * ng, n[0] + 2 * ng)
        u = u.to(dt).contiguous()
        inner = u.double() if ng == 0 else u[:, ng:-ng, ng:-ng, ng:-ng].double()
        got = dict(u=u, dx=dx, ng=ng, dt=_signal_dt([_prim(inner)], dx))
        if kind == "adjoint":
            g = _gen(seed + 77)
            got["lam"] = torch.randn(inner.shape, generator=g, device="cuda", dtype=torch.float64)
            nf = 10 * (n[2] * n[1] + n[2] * n[0] + n[1] * n[0])
            got["lam_bflux"] = (torch.randn(nf, generator=g, device="cuda", dtype=torch.float64)
                                * got["dt"] / dx if case["bflux"] else None)
        return got
    if kind == "batch":
        dims, ng, dx = _batch_dims(case), case["ng"], 1.0 / 256
        u = _shocked(seed, dims, ng, dx).to(dt)
        at, _, _ = _offsets(dims, ng)
        cells = []
        for n, ids in _groups(dims):
            cells.append(_prim(_gather(u, at[0], ids, n, ng)[..., ng:-ng, ng:-ng, ng:-ng].double()))
        return dict(u=u, dx=dx, ng=ng, dims=dims, dt=_signal_dt(cells, dx))
    if kind == "rollout":
        u, dx = _smooth(seed, case["n"])
        g = _gen(seed + 77)
        return dict(u=u, dx=dx, dt=_signal_dt([_prim(u)], dx),
                    lam=torch.randn(u.shape, generator=g, device="cuda", dtype=torch.float64))
    if kind == "mhd":
        u, dx = _turbulence(seed, case["nx"], case["ny"], case["nz"], mach=1.0, beta=100.0)
        u = u.to(dt).contiguous()
        s, ch = _mhd_speeds(_mhd_prim(u.double()))
        return dict(u=u, dx=dx, dt=0.4 * dx / s, ch=ch)
    lo, size = _hierarchy(case)
    coarse, full = _hierarchy_state(seed, case)
    coarse = coarse.to(dt).contiguous()
    at, _, _ = _offsets(2 * size, 2)
    fine = torch.zeros(at[1], dtype=dt, device="cuda")
    for o, a, s in zip(at[0], lo, size):
        e = 2 * s + 4
        box = fine[o:o + 5 * int(np.prod(e))].view(5, e[2], e[1], e[0])
        b, t = 2 * a, 2 * (a + s)
        box[:, 2:-2, 2:-2, 2:-2] = full[:, b[2]:t[2], b[1]:t[1], b[0]:t[0]]
    dxc = 1.0 / case["nc"]
    # same dt on both levels: that of the finer one
    return dict(coarse=coarse, fine=fine, lo=lo, size=size, dx=dxc,
                dt=_signal_dt([_prim(coarse.double())], dxc / 2) * 0.95)


# ---------------------------------------------------------------- a pass

def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind = case["kind"]
    s["dt_dev"] = _scalar(s["dt"])
    s["dt_next"] = torch.zeros(1, dtype=torch.float64, device="cuda")
    if kind == "step" and case["reuse"]:
        n = (case["nx"], case["ny"], case["nz"])
        s["out"] = torch.zeros((5,) + n[::-1], dtype=s["u"].dtype, device="cuda")
        s["bflux"] = (torch.zeros(godunov.bflux_size(*n), dtype=s["u"].dtype, device="cuda")
                      if case["bflux"] else None)
    elif kind == "batch":
        i, o, f = _offsets(s["dims"], s["ng"])
        s["table"] = godunov.patch_table(s["dims"], s["ng"], i[0], o[0], f[0], s["dx"])
        s["out"] = torch.zeros(o[1], dtype=s["u"].dtype, device="cuda")
        s["bflux"] = torch.zeros(f[1], dtype=s["u"].dtype, device="cuda")
    elif kind == "mhd":
        s["out"] = torch.zeros_like(s["u"])
        s["ch_dev"] = _scalar(s["ch"])
        s["ch_next"] = torch.zeros(1, dtype=torch.float64, device="cuda")
    elif kind == "adjoint":
        s["out"] = torch.zeros_like(s["u"])
    elif kind == "amr":
        i, o, f = _offsets(2 * s["size"], 2)
        table = godunov.amr_patch_table(s["lo"], 2 * s["size"], i[0], o[0], f[0])
        s["plan"] = godunov.AmrPlan((case["nc"],) * 3, s["dx"], table)
        s["coarse_out"] = torch.zeros_like(s["coarse"])
        s["fine_out"] = torch.zeros(o[1], dtype=s["fine"].dtype, device="cuda")
        s["flux"] = torch.zeros(f[1], dtype=s["fine"].dtype, device="cuda")
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "step":
        opts = dict(ng=s["ng"], periodic=s["ng"] == 0, limiter=c["limiter"], riemann=c["riemann"],
                    want_bflux=c["bflux"])
        if c["reuse"]:
            opts.update(out=s["out"], bflux=s["bflux"])
        dt = s["dt_dev"]
        if c["cfl"] == "before":
            dt = godunov.cfl_dt(s["u"], GAMMA, s["dx"], CFL, ng=s["ng"], periodic=s["ng"] == 0)
        if c["cfl"] == "fused":
            opts.update(cfl=CFL, dt_next=s["dt_next"])
        out, bflux = godunov.step(s["u"], GAMMA, s["dx"], dt_dev=dt, **opts)
        return {"u": out, "bflux": bflux, "dt": {"before": dt, "fused": s["dt_next"]}.get(c["cfl"])}
    if kind == "batch":
        opts = dict(cfl=CFL, dt_next=s["dt_next"]) if c["cfl"] == "fused" else {}
        out, bflux = godunov.step_batched(s["u"], s["table"], GAMMA, out=s["out"], bflux=s["bflux"],
                                          dt_dev=s["dt_dev"], limiter=c["limiter"],
                                          riemann=c["riemann"], **opts)
        return {"u": out, "bflux": bflux, "dt": s["dt_next"] if opts else None}
    if kind == "adjoint":
        return godunov.step_adjoint(s["u"], s["lam"], GAMMA, s["dx"], s["dt"],
                                    lam_bflux=s["lam_bflux"], ng=2, periodic=c["periodic"],
                                    limiter=c["limiter"], riemann=c["riemann"], out=s["out"])
    if kind == "rollout":
        u0 = s["u"].detach().requires_grad_(True)
        u = godunov.rollout(u0, GAMMA, s["dx"], s["dt"], c["nsteps"], c["every"], c["limiter"],
                            c["riemann"])
        grad, = torch.autograd.grad(u, u0, s["lam"])
        return {"u": u.detach(), "grad": grad}
    if kind == "mhd":
        out = godunov.step_mhd(s["u"], GAMMA, s["dx"], dt_dev=s["dt_dev"], ch_dev=s["ch_dev"],
                               limiter=c["limiter"], out=s["out"], cfl=0.4, dt_next=s["dt_next"],
                               ch_next=s["ch_next"])
        return {"u": out, "dt": s["dt_next"], "ch": s["ch_next"]}
    co, fo, fl = s["plan"].step(s["coarse"], s["fine"], GAMMA, dt_dev=s["dt_dev"],
                                coarse_out=s["coarse_out"], fine_out=s["fine_out"],
                                fine_flux=s["flux"], limiter=c["limiter"], riemann=c["riemann"])
    return {"coarse": co, "fine": fo, "flux": fl, "ghosted": s["fine"]}


def work(case):
    """Bytes: the state (for a patch the cells its stencils reach) read once,
    what the call returns written once; a rollout's steps depend on one
    another, so each counts. Operations: those of the scheme's formulas per
    cell, each face solved once (an add, a multiply or a fused pair is one)."""
    b = 4 if case.get("dtype") == "f32" else 8
    kind = case["kind"]

    def read(n, deep):
        x, y, z = (int(v) for v in n)
        return x * y * z + 2 * deep * (x * y + y * z + z * x) + 4 * (deep - 1) ** 2 * (x + y + z)

    def flux(n):
        return 10 * (n[0] * n[1] + n[1] * n[2] + n[2] * n[0])

    ops = 800 if case["limiter"].startswith("ppm") else 420
    if kind == "step":
        n = (case["nx"], case["ny"], case["nz"])
        cells = n[0] * n[1] * n[2]
        deep = 3 if case["limiter"].startswith("ppm") else 2
        got = cells if case["init"] == "turbulence" else read(n, deep)
        return {"bytes": b * (5 * got + 5 * cells + (flux(n) if case["bflux"] else 0)),
                "flops": ops * cells}
    if kind == "batch":
        dims = _batch_dims(case)
        deep = 3 if case["limiter"].startswith("ppm") else 2
        cells = sum(int(np.prod(n)) for n in dims)
        total = sum(5 * read(n, deep) + int(flux(n)) for n in dims) + 5 * cells
        return {"bytes": b * total, "flops": ops * cells}
    if kind == "adjoint":
        n = (case["nx"], case["ny"], case["nz"])
        cells = n[0] * n[1] * n[2]
        box = cells if case["periodic"] else read(n, 2)
        return {"bytes": 8 * (10 * box + 5 * cells + (flux(n) if case["bflux"] else 0)),
                "flops": 1100 * cells}
    if kind == "rollout":
        cells = case["n"] ** 3
        return {"bytes": 8 * case["nsteps"] * 25 * cells, "flops": 1520 * case["nsteps"] * cells}
    if kind == "mhd":
        cells = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": b * 18 * cells, "flops": 1400 * cells}
    _, size = _hierarchy(case)
    fine = sum(int(np.prod(2 * s)) for s in size)
    ghosts = sum(int(np.prod(2 * s + 4)) for s in size) - fine
    faces = sum(int(flux(2 * s)) for s in size)
    coarse = case["nc"] ** 3
    return {"bytes": b * (10 * coarse + 10 * fine + 5 * ghosts + faces),
            "flops": 420 * (coarse + fine)}


# ---------------------------------------------------------------- in 64 bits
# A state is a list of tensors [..., z, y, x]; axis d = 0, 1, 2 is x, y, z.

def _extend(u, g, mode="wrap"):
    """u with g more cells on every side of its last three axes."""
    for ax in (-1, -2, -3):
        n = u.shape[ax]
        i = torch.arange(-g, n + g, device=u.device)
        u = u.index_select(u.dim() + ax, i % n if mode == "wrap" else i.clamp(0, n - 1))
    return u


def _cut(a, d, lo, hi):
    """a without its first lo and last hi cells along axis d."""
    return a.narrow(a.dim() - 1 - d, lo, a.shape[-1 - d] - lo - hi)


def _inner(a, g, but=None):
    for d in range(3):
        if d != but:
            a = _cut(a, d, g, g)
    return a


def _prim(U):
    U = U.unbind(-4)
    rho = U[0].clamp(min=FLOOR)
    u, v, w = U[1] / rho, U[2] / rho, U[3] / rho
    p = (GAMMA - 1.0) * (U[4] - 0.5 * (U[1] * u + U[2] * v + U[3] * w))
    return [rho, u, v, w, p.clamp(min=FLOOR)]


def _slope(a, b, limiter):
    if limiter == "unlimited":
        return 0.5 * (a + b)
    same = ((a > 0) & (b > 0)) | ((a < 0) & (b < 0))
    if limiter == "minmod":
        s = torch.where(a.abs() <= b.abs(), a, b)
    else:
        two = torch.where(a.abs() <= b.abs(), 2 * a, 2 * b)
        mid = 0.5 * (a + b)
        s = torch.where(two.abs() <= mid.abs(), two, mid)
    return torch.where(same, s, torch.zeros_like(s))


def _edges(a, d):
    """Limited parabola edges along d for the cells three in from each end."""
    dif = _cut(a, d, 1, 0) - _cut(a, d, 0, 1)
    da = _slope(_cut(dif, d, 0, 1), _cut(dif, d, 1, 0), "mc")
    a1 = _cut(a, d, 1, 1)
    face = 0.5 * (_cut(a1, d, 0, 1) + _cut(a1, d, 1, 0)) - (_cut(da, d, 1, 0) - _cut(da, d, 0, 1)) / 6
    lo, hi, a0 = _cut(face, d, 0, 1), _cut(face, d, 1, 0), _cut(a, d, 2, 2)
    flat = (hi - a0) * (a0 - lo) <= 0
    D, m = hi - lo, a0 - 0.5 * (lo + hi)
    new_lo = torch.where(D * m > D * D / 6, 3 * a0 - 2 * hi, lo)
    new_hi = torch.where(D * m < -D * D / 6, 3 * a0 - 2 * lo, hi)
    return torch.where(flat, a0, new_lo), torch.where(flat, a0, new_hi)


def _hllc(L, R, riemann):
    """Flux from rotated states (rho, u_n, u_t1, u_t2, p)."""
    def cons(W):
        E = W[4] / (GAMMA - 1) + 0.5 * W[0] * (W[1] ** 2 + W[2] ** 2 + W[3] ** 2)
        U = [W[0], W[0] * W[1], W[0] * W[2], W[0] * W[3], E]
        return U, [U[1], U[1] * W[1] + W[4], U[2] * W[1], U[3] * W[1], W[1] * (E + W[4])]

    (UL, FL), (UR, FR) = cons(L), cons(R)
    cL, cR = torch.sqrt(GAMMA * L[4] / L[0]), torch.sqrt(GAMMA * R[4] / R[0])
    a, b = L[1] - cL, R[1] - cR
    SL = torch.where(a <= b, a, b)
    a, b = L[1] + cL, R[1] + cR
    SR = torch.where(a >= b, a, b)
    supL, supR = SL >= 0, SR <= 0
    if riemann == "hll":
        return [torch.where(supL, fl, torch.where(supR, fr, (SR * fl - SL * fr + SL * SR * (ur - ul))
                                                  / (SR - SL)))
                for fl, fr, ul, ur in zip(FL, FR, UL, UR)]
    mL, mR = L[0] * (SL - L[1]), R[0] * (SR - R[1])
    S = (R[4] - L[4] + mL * L[1] - mR * R[1]) / (mL - mR)
    F = []
    for W, U, FK, SK, m in ((L, UL, FL, SL, mL), (R, UR, FR, SR, mR)):
        f = m / (SK - S)
        e = U[4] / W[0] + (S - W[1]) * (S + W[4] / m)
        F.append([FK[q] + SK * (f * s - U[q]) for q, s in enumerate((1.0, S, W[2], W[3], e))])
    left = S >= 0
    return [torch.where(supL, FL[q], torch.where(left, F[0][q], torch.where(supR, FR[q], F[1][q])))
            for q in range(5)]


def _godunov(U, g, c, limiter, riemann):
    """New interior state and the face fluxes along x, y, z of the ghosted
    state U [..., 5, z, y, x] with g ghost layers; c = dt/dx."""
    ppm = limiter.startswith("ppm")
    W = [_inner(w, g - (3 if ppm else 2)) for w in _prim(U)]
    r = 3 if ppm else 2
    C = [_inner(w, r - 1) for w in W]                       # the cells whose states faces need
    lo, hi, S = [], [], []
    for d in range(3):
        ld, hd, sd = [], [], []
        for q in range(5):
            w = _inner(W[q], r - 1, but=d)
            if ppm:
                el, eh = _edges(w, d)
                ld.append(el - C[q]), hd.append(eh - C[q]), sd.append(eh - el)
            else:
                dif = _cut(w, d, 1, 0) - _cut(w, d, 0, 1)
                s = _slope(_cut(dif, d, 0, 1), _cut(dif, d, 1, 0), limiter)
                ld.append(-0.5 * s), hd.append(0.5 * s), sd.append(s)
        lo.append(ld), hi.append(hd), S.append(sd)

    def term(d):                                            # A_d(W) S_d
        t = [C[1 + d] * S[d][q] for q in range(5)]
        t[0] = t[0] + C[0] * S[d][1 + d]
        t[1 + d] = t[1 + d] + S[d][4] / C[0]
        t[4] = t[4] + GAMMA * C[4] * S[d][1 + d]
        return t

    T = [term(d) for d in range(3)]
    cs = torch.sqrt(GAMMA * C[4] / C[0])
    flux = []
    for d in range(3):
        n, t1, t2 = 1 + d, 1 + (d + 1) % 3, 1 + (d + 2) % 3
        if limiter == "ppm_ct":
            others = [e for e in range(3) if e != d]
            base = [C[q] - 0.5 * c * (T[others[0]][q] + T[others[1]][q]) for q in range(5)]
            a6 = [-3 * (lo[d][q] + hi[d][q]) for q in range(5)]

            def traced(upper):
                got = list(hi[d]) if upper else list(lo[d])
                for w, speed in enumerate((C[n] - cs, C[n], C[n] + cs)):
                    s = speed * c
                    on = (s > 0) if upper else (s < 0)
                    sg = -1.0 if upper else 1.0
                    off = [-0.5 * s * (S[d][q] + sg * (1 + sg * s * 2 / 3) * a6[q]) for q in range(5)]
                    if w == 1:
                        add = {0: off[0] - off[4] / cs ** 2, t1: off[t1], t2: off[t2]}
                    else:
                        k = -1.0 if w == 0 else 1.0
                        beta = k * C[0] / (2 * cs) * off[n] + off[4] / (2 * cs ** 2)
                        add = {0: beta, n: k * cs / C[0] * beta, 4: cs ** 2 * beta}
                    for q, v in add.items():
                        got[q] = got[q] + torch.where(on, v, torch.zeros_like(v))
                return got

            down, up = ([base[q] + e[q] for q in range(5)] for e in (traced(False), traced(True)))
        else:
            base = [C[q] - 0.5 * c * (T[0][q] + T[1][q] + T[2][q]) for q in range(5)]
            down, up = ([base[q] + e[d][q] for q in range(5)] for e in (lo, hi))
        for st in (down, up):
            st[0], st[4] = st[0].clamp(min=FLOOR), st[4].clamp(min=FLOOR)
        order = [0, n, t1, t2, 4]
        L = [_cut(_inner(up[q], 1, but=d), d, 0, 1) for q in order]
        R = [_cut(_inner(down[q], 1, but=d), d, 1, 0) for q in order]
        F = _hllc(L, R, riemann)
        flux.append([F[order.index(q)] for q in range(5)])
    old = _inner(U, g).unbind(-4)
    new = [old[q] - c * sum(_cut(flux[d][q], d, 1, 0) - _cut(flux[d][q], d, 0, 1) for d in range(3))
           for q in range(5)]
    return torch.stack(new, -4), flux


def _sheets(flux):
    """The six boundary sheets of one or several patches, flat per patch."""
    parts = []
    for d in range(3):
        F = torch.stack(flux[d], -4)
        ax = F.dim() - 1 - d
        for at in (0, F.shape[ax] - 1):
            parts.append(F.select(ax, at).flatten(-3))
    return torch.cat(parts, -1)


def _groups(dims):
    by = {}
    for i, n in enumerate(dims):
        by.setdefault(tuple(int(v) for v in n), []).append(i)
    return by.items()


def _gather(flat, at, ids, n, ng):
    e = [v + 2 * ng for v in n]
    size = 5 * e[0] * e[1] * e[2]
    i = torch.as_tensor(at[ids], device=flat.device)[:, None] + torch.arange(size, device=flat.device)
    return flat[i].view(len(ids), 5, e[2], e[1], e[0])


def _scatter(flat, at, ids, values):
    v = values.flatten(1)
    i = torch.as_tensor(at[ids], device=flat.device)[:, None] + torch.arange(v.shape[1], device=flat.device)
    flat[i] = v


def _mhd_prim(U):
    rho = U[0].clamp(min=FLOOR)
    u, v, w = U[1] / rho, U[2] / rho, U[3] / rho
    p = (GAMMA - 1) * (U[4] - 0.5 * (U[1] * u + U[2] * v + U[3] * w)
                       - 0.5 * (U[5] ** 2 + U[6] ** 2 + U[7] ** 2))
    return [rho, u, v, w, p.clamp(min=FLOOR), U[5], U[6], U[7], U[8]]


def _mhd_cons(W):
    E = (W[4] / (GAMMA - 1) + 0.5 * W[0] * (W[1] ** 2 + W[2] ** 2 + W[3] ** 2)
         + 0.5 * (W[5] ** 2 + W[6] ** 2 + W[7] ** 2))
    return [W[0], W[0] * W[1], W[0] * W[2], W[0] * W[3], E, W[5], W[6], W[7], W[8]]


def _fast(W, bn):
    a2 = GAMMA * W[4] / W[0]
    s = a2 + (W[5] ** 2 + W[6] ** 2 + W[7] ** 2) / W[0]
    return torch.sqrt(0.5 * (s + torch.sqrt((s * s - 4 * a2 * bn * bn / W[0]).clamp(min=0))))


def _mhd_speeds(W):
    v = [W[1 + d].abs() + _fast(W, W[5 + d]) for d in range(3)]
    return float((v[0] + v[1] + v[2]).max()), float(max(x.max() for x in v))


def _mhd_flux(W, d, ch):
    un, Bn = W[1 + d], W[5 + d]
    pT = W[4] + 0.5 * (W[5] ** 2 + W[6] ** 2 + W[7] ** 2)
    uB = W[1] * W[5] + W[2] * W[6] + W[3] * W[7]
    U = _mhd_cons(W)
    F = [U[0] * un, *[U[1 + k] * un - Bn * W[5 + k] + (pT if k == d else 0.0) for k in range(3)],
         (U[4] + pT) * un - Bn * uB,
         *[W[8] if k == d else un * W[5 + k] - W[1 + k] * Bn for k in range(3)], ch * ch * Bn]
    return F


def _hlld(L, R, d, ch):
    """GLM + HLLD flux along d (Miyoshi & Kusano 2005)."""
    t1, t2 = (d + 1) % 3, (d + 2) % 3
    Bn = 0.5 * (L[5 + d] + R[5 + d]) - (R[8] - L[8]) / (2 * ch)
    psi = 0.5 * (L[8] + R[8]) - 0.5 * ch * (R[5 + d] - L[5 + d])
    order = [0, 1 + d, 1 + t1, 1 + t2, 4, 5 + d, 5 + t1, 5 + t2]
    side = []
    for W in (L, R):
        w = [W[q] for q in order]
        w[5] = Bn
        w.append(psi)
        U, F = _mhd_cons(w), _mhd_flux(w, 0, ch)
        side.append((w, U, F, w[4] + 0.5 * (w[5] ** 2 + w[6] ** 2 + w[7] ** 2), _fast(w, Bn)))
    (wl, Ul, Fl, pl, cl), (wr, Ur, Fr, pr, cr) = side
    SL, SR = torch.minimum(wl[1] - cl, wr[1] - cr), torch.maximum(wl[1] + cl, wr[1] + cr)
    dL, dR = (SL - wl[1]) * wl[0], (SR - wr[1]) * wr[0]
    SM = (dR * wr[1] - dL * wl[1] - pr + pl) / (dR - dL)
    pS = (dR * pl - dL * pr + dL * dR * (wr[1] - wl[1])) / (dR - dL)
    star = []
    for (w, U, F, pT, _), S in ((side[0], SL), (side[1], SR)):
        rs = w[0] * (S - w[1]) / (S - SM)
        den = w[0] * (S - w[1]) * (S - SM) - Bn * Bn
        top = w[0] * (S - w[1]) ** 2
        bad = den.abs() <= 1e-12 * (top + Bn * Bn)
        iden = torch.where(bad, torch.zeros_like(den), 1 / torch.where(bad, torch.ones_like(den), den))
        t = Bn * (SM - w[1]) * iden
        f = torch.where(bad, torch.ones_like(den), (top - Bn * Bn) * iden)
        v, z, By, Bz = w[2] - w[6] * t, w[3] - w[7] * t, w[6] * f, w[7] * f
        uB = w[1] * Bn + w[2] * w[6] + w[3] * w[7]
        uBs = SM * Bn + v * By + z * Bz
        Es = ((S - w[1]) * U[4] - pT * w[1] + pS * SM + Bn * (uB - uBs)) / (S - SM)
        star.append(([rs, rs * SM, rs * v, rs * z, Es, Bn, By, Bz], v, z, torch.sqrt(rs), uBs))
    (sl, vl, zl, ql, bl), (sr, vr, zr, qr, br) = star
    sg = torch.sign(Bn)
    v = (ql * vl + qr * vr + (sr[6] - sl[6]) * sg) / (ql + qr)
    z = (ql * zl + qr * zr + (sr[7] - sl[7]) * sg) / (ql + qr)
    By = (ql * sr[6] + qr * sl[6] + ql * qr * (vr - vl) * sg) / (ql + qr)
    Bz = (ql * sr[7] + qr * sl[7] + ql * qr * (zr - zl) * sg) / (ql + qr)
    uB = SM * Bn + v * By + z * Bz
    flux = []
    for (w, U, F, _, _), S, (us, _, _, q, b), k in ((side[0], SL, star[0], -1.0), (side[1], SR, star[1], 1.0)):
        Sa = SM + k * Bn.abs() / q
        uss = [us[0], us[1], us[0] * v, us[0] * z, us[4] + k * q * (b - uB) * sg, Bn, By, Bz]
        f1 = [F[i] + S * (us[i] - U[i]) for i in range(8)]
        outside = (Sa >= 0) if k < 0 else (Sa <= 0)
        flux.append([torch.where(outside, f1[i], f1[i] + Sa * (uss[i] - us[i])) for i in range(8)])
    got = [torch.where(SL >= 0, Fl[i], torch.where(SR <= 0, Fr[i], torch.where(SM >= 0, flux[0][i], flux[1][i])))
           for i in range(8)]
    out = [None] * 9
    for i, q in enumerate(order):
        out[q] = got[i]
    out[5 + d], out[8] = psi, ch * ch * Bn
    return out


def _mhd(u, c, ch, damp, limiter):
    U = _extend(u, 2)
    W = _mhd_prim(U)
    C = [_inner(w, 1) for w in W]
    S = []
    for d in range(3):
        sd = []
        for w in W:
            dif = _inner(w, 1, but=d)
            dif = _cut(dif, d, 1, 0) - _cut(dif, d, 0, 1)
            sd.append(_slope(_cut(dif, d, 0, 1), _cut(dif, d, 1, 0), limiter))
        S.append(sd)
    faces, dU = [], [torch.zeros_like(C[0]) for _ in range(9)]
    for d in range(3):
        pair = []
        for sg in (0.5, -0.5):
            w = [a + sg * s for a, s in zip(C, S[d])]
            w[0], w[4] = w[0].clamp(min=FLOOR), w[4].clamp(min=FLOOR)
            pair.append(w)
        faces.append(pair)
        Fu, Fd = _mhd_flux(pair[0], d, ch), _mhd_flux(pair[1], d, ch)
        dU = [x - 0.5 * c * (a - b) for x, a, b in zip(dU, Fu, Fd)]
    new = list(_inner(U, 2).unbind(0))
    for d in range(3):
        up, dn = ([q + x for q, x in zip(_mhd_cons(w), dU)] for w in faces[d])
        L = [_cut(_inner(a, 1, but=d), d, 0, 1) for a in _mhd_prim(up)]
        R = [_cut(_inner(a, 1, but=d), d, 1, 0) for a in _mhd_prim(dn)]
        F = _hlld(L, R, d, ch)
        new = [n - c * (_cut(f, d, 1, 0) - _cut(f, d, 0, 1)) for n, f in zip(new, F)]
    new[8] = new[8] * damp
    return torch.stack(new)


def _amr(s, case):
    """The two-level step on full grids of both levels: outside the patches
    the fine grid holds the prolongation that fills their ghosts."""
    nc, lo, size = case["nc"], s["lo"], s["size"]
    coarse, c = s["coarse"].double(), s["dt"] / s["dx"]
    E = _extend(coarse, 1)
    child = torch.arange(2 * nc, device="cuda")
    par, sg = child // 2, 2.0 * (child % 2) - 1.0
    slope = []
    for d in range(3):
        w = _inner(E, 1, but=d)
        dif = _cut(w, d, 1, 0) - _cut(w, d, 0, 1)
        slope.append(_slope(_cut(dif, d, 0, 1), _cut(dif, d, 1, 0), "minmod"))

    def spread(a):
        return a[:, par][:, :, par][:, :, :, par]

    fine = spread(coarse) + 0.25 * (spread(slope[0]) * sg + spread(slope[1]) * sg[:, None]
                                    + spread(slope[2]) * sg[:, None, None])
    at, out_at, fl_at = _offsets(2 * size, 2)
    covered = torch.zeros((nc, nc, nc), dtype=torch.bool, device="cuda")
    for o, a, n in zip(at[0], lo, size):
        e, b, t = 2 * n + 4, 2 * a, 2 * (a + n)
        box = s["fine"][o:o + 5 * int(np.prod(e))].view(5, e[2], e[1], e[0])
        fine[:, b[2]:t[2], b[1]:t[1], b[0]:t[0]] = box[:, 2:-2, 2:-2, 2:-2].double()
        covered[a[2]:a[2] + n[2], a[1]:a[1] + n[1], a[0]:a[0] + n[0]] = True
    ghosted = torch.empty(at[1], dtype=torch.float64, device="cuda")
    fine_out = torch.empty(out_at[1], dtype=torch.float64, device="cuda")
    sheets = torch.empty(fl_at[1], dtype=torch.float64, device="cuda")
    new, Ff = _godunov(_extend(fine, 2), 2, 2 * c, case["limiter"], case["riemann"])
    Ff = [torch.stack(f) for f in Ff]
    for k, (a, n) in enumerate(zip(lo, size)):
        b, t = 2 * a, 2 * (a + n)
        ghosted[at[0][k]:at[0][k] + 5 * int(np.prod(2 * n + 4))] = _wrap_box(fine, b - 2, t + 2).reshape(-1)
        fine_out[out_at[0][k]:out_at[0][k] + 5 * int(np.prod(2 * n))] = (
            new[:, b[2]:t[2], b[1]:t[1], b[0]:t[0]].reshape(-1))
        parts = []
        for d in range(3):
            for x in (b[d], t[d]):
                f = Ff[d].select(3 - d, int(x))
                i, j = [ax for ax in (2, 1, 0) if ax != d]          # slow, fast
                parts.append(f[:, b[i]:t[i], b[j]:t[j]].reshape(-1))
        v = torch.cat(parts)
        sheets[fl_at[0][k]:fl_at[0][k] + len(v)] = v
    old = _extend(coarse, 2)
    _, Fc = _godunov(old, 2, c, case["limiter"], case["riemann"])
    out = coarse.clone()
    for d in range(3):
        F = torch.stack(Fc[d])
        left = torch.roll(covered, 1, dims=2 - d)
        seam = torch.cat([left ^ covered, (left ^ covered).narrow(2 - d, 0, 1)], dim=2 - d)
        f = Ff[d].index_select(3 - d, 2 * torch.arange(nc + 1, device="cuda"))
        for ax in (1, 2, 3):
            if ax != 3 - d:
                f = 0.5 * (f.index_select(ax, 2 * torch.arange(nc, device="cuda"))
                           + f.index_select(ax, 2 * torch.arange(nc, device="cuda") + 1))
        F = torch.where(seam, f, F)
        out = out - c * (_cut(F, d, 1, 0) - _cut(F, d, 0, 1))
    mean = new.view(5, nc, 2, nc, 2, nc, 2).mean(dim=(2, 4, 6))
    return {"coarse": torch.where(covered, mean, out), "fine": fine_out, "flux": sheets,
            "ghosted": ghosted}


def _wrap_box(a, lo, hi):
    for ax in range(3):
        n = a.shape[3 - ax]
        a = a.index_select(3 - ax, torch.arange(int(lo[ax]), int(hi[ax]), device=a.device) % n)
    return a


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    opts = (case["limiter"], case.get("riemann", "hllc"))
    if kind == "step":
        u, g = s["u"].double(), s["ng"]
        if g == 0:
            g = 3
            u = _extend(u, g)
        new, flux = _godunov(u, g, s["dt"] / s["dx"], *opts)
        dt = {"before": s["dt"], "fused": _signal_dt([_prim(new)], s["dx"])}.get(case["cfl"])
        return {"u": new, "bflux": _sheets(flux) if case["bflux"] else None,
                "dt": None if dt is None else _scalar(dt)}
    if kind == "batch":
        at, out_at, fl_at = _offsets(s["dims"], s["ng"])
        out = torch.empty(out_at[1], dtype=torch.float64, device="cuda")
        bflux = torch.empty(fl_at[1], dtype=torch.float64, device="cuda")
        cells = []
        for n, ids in _groups(s["dims"]):
            new, flux = _godunov(_gather(s["u"], at[0], ids, n, s["ng"]).double(), s["ng"],
                                 s["dt"] / s["dx"], *opts)
            _scatter(out, out_at[0], ids, new)
            _scatter(bflux, fl_at[0], ids, _sheets(flux))
            cells.append(_prim(new))
        dt = _scalar(_signal_dt(cells, s["dx"])) if case["cfl"] == "fused" else None
        return {"u": out, "bflux": bflux, "dt": dt}
    if kind == "adjoint":
        u = s["u"].clone().requires_grad_(True)
        new, flux = _godunov(_extend(u, 2) if case["periodic"] else u, 2, s["dt"] / s["dx"], *opts)
        total = (new * s["lam"]).sum()
        if s["lam_bflux"] is not None:
            total = total + (_sheets(flux) * s["lam_bflux"]).sum()
        return torch.autograd.grad(total, u)[0]
    if kind == "rollout":
        states = [s["u"]]
        for _ in range(case["nsteps"]):
            states.append(_godunov(_extend(states[-1], 2), 2, s["dt"] / s["dx"], *opts)[0])
        lam = s["lam"]
        for st in reversed(states[:-1]):
            st = st.clone().requires_grad_(True)
            new, _ = _godunov(_extend(st, 2), 2, s["dt"] / s["dx"], *opts)
            lam, = torch.autograd.grad(new, st, lam)
        return {"u": states[-1], "grad": lam}
    if kind == "mhd":
        c, ch = s["dt"] / s["dx"], s["ch"]
        new = _mhd(s["u"].double(), c, ch, math.exp(-0.1 * ch * c), case["limiter"])
        sm, ch_next = _mhd_speeds(_mhd_prim(new))
        return {"u": new, "dt": _scalar(0.4 * s["dx"] / sm), "ch": _scalar(ch_next)}
    return _amr(s, case)
