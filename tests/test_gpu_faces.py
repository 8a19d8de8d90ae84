"""Faces outside the Riemann fan.

A face whose fan lies wholly to one side has the physical flux of the state on the
other side. States are made of few-bit numbers (densities powers of two, gamma
1.5), so that every product and sum of that flux is exact in double precision, and
slopes vanish, so the faces see the cells' own states."""
import numpy as np
import pytest

from helpers import say

pytestmark = pytest.mark.gpu
G = 1.5


@pytest.fixture(scope="module")
def gd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1412_0934_amd import godunov
    return godunov


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


P_FLOOR = 1e-40


def sheet(b, axis, side, n):
    """One sheet [5][...] of a boundary-flux buffer of a cube of n cells."""
    at = (2 * axis + side) * 5 * n * n
    return b[at:at + 5 * n * n].reshape(5, n * n)


@pytest.mark.parametrize("lim", ["minmod", "mc", "ppm", "ppm_ct"])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("cold", [False, True])
def test_supersonic_face_has_the_upwind_flux(gd, lim, axis, cold):
    """The boundary fluxes of uniform patches, to the two roundings that a product
    of three factors or a product and a sum may take where they are not exact.
    Cold: no pressure but the floor's, and a sound speed below the last place of
    the velocity, so that no wave speed differs from it."""
    n, ng = 3, 3
    rng = np.random.default_rng(axis)
    say("supersonic faces", lim, axis, "cold" if cold else "warm")
    for _ in range(12):
        rho = 2.0 ** rng.integers(-2, 3)
        p = 0.0 if cold else rho * rng.integers(16, 64) / 4.0           # c^2 of 6 to 24
        vel = rng.integers(-64, 64, 3) / 16.0
        vel[axis] = rng.choice([-1, 1]) * rng.integers(256, 512) / 8.0
        E = 2.0 * p + 0.5 * rho * (vel @ vel)
        U = np.array([rho, *(rho * vel), E])
        F = vel[axis] * np.array([rho, *(rho * vel), E + p])
        F[1 + axis] += p
        u = dev(np.broadcast_to(U.reshape(5, 1, 1, 1), (5,) + (n + 2 * ng,) * 3))
        _, b = gd.step(u, G, 1 / 16, 1 / 1024, ng=ng, limiter=lim, rho_floor=P_FLOOR, p_floor=P_FLOOR)
        for side in (0, 1):
            got = sheet(host(b), axis, side, n)
            assert (np.abs(got - F[:, None]) <= 2 * np.spacing(np.abs(F))[:, None]).all(), (U, got, F)


@pytest.mark.parametrize("lim", ["minmod", "ppm"])
def test_gas_without_pressure_or_floor_is_no_number(gd, lim):
    """With a zero floor a gas without pressure has no sound speed and no upwind
    side: its fluxes are NaN, not those of whichever side comes last."""
    n, ng = 3, 3
    rho = np.full((n + 2 * ng,) * 3, 2.0)
    u = np.stack([rho, 4.0 * rho, 0.0 * rho, 0.0 * rho, 8.0 * rho])
    say("no pressure", lim)
    _, b = gd.step(dev(u), G, 1 / 16, 1 / 1024, ng=ng, limiter=lim, rho_floor=0.0, p_floor=0.0)
    assert np.isnan(sheet(host(b), 0, 0, n)).all()
    lam = np.ones((5, n, n, n))
    got = host(gd.step_adjoint(dev(u), dev(lam), G, 1 / 16, 1 / 1024, ng=ng, rho_floor=0.0,
                               p_floor=0.0))
    assert not np.isfinite(got[:, ng:-ng, ng:-ng, ng:-ng]).all()


def rotate(v, axis, fields=((1, 2, 3),)):
    """Variables of data along x turned to an axis (cyclically)."""
    v = np.array(v)
    for f in fields:
        v[[f[(c + axis) % 3] for c in range(3)]] = v[list(f)]
    return v


def along(profile, axis, shape=(4, 4)):
    """A profile [var][i] as a box [var][z][y][x] that varies along one axis only."""
    nvar, n = profile.shape
    dims = [shape[1], shape[0]]
    dims.insert(2 - axis, n)                    # z, y, x
    one = [1, 1, 1]
    one[2 - axis] = n
    return np.ascontiguousarray(np.broadcast_to(profile.reshape([nvar] + one), [nvar] + dims))


def mhd_blocks(sign, cold, seed, n=32):
    """n MHD states in blocks of two cells, the flow faster than any wave along the
    axis and the field along it uniform: (U, F), [9][2n] each. Cold: a weak field
    too, so that the fast speed lies below the last place of the velocity."""
    rng = np.random.default_rng(seed)
    rho = 2.0 ** rng.integers(-2, 3, n)
    u = sign * rng.integers(256, 512, n) / 8.0
    v, w = np.zeros(n), np.zeros(n)
    p = np.zeros(n) if cold else rho * rng.integers(16, 64, n) / 4.0
    weak = 2.0 ** -60 if cold else 1.0
    Bx = np.full(n, weak)
    By, Bz = (weak * rng.integers(-16, 16, n) / 8.0 for _ in range(2))
    psi = np.zeros(n)
    B2 = Bx * Bx + By * By + Bz * Bz
    E = 2.0 * p + 0.5 * rho * u * u + 0.5 * B2
    pT = p + 0.5 * B2
    U = np.stack([rho, rho * u, rho * v, rho * w, E, Bx, By, Bz, psi])
    F = np.stack([rho * u, rho * u * u + pT - Bx * Bx, -Bx * By, -Bx * Bz,
                  (E + pT) * u - Bx * (u * Bx), 0.0 * u, u * By, u * Bz, CH * CH * Bx])
    return np.repeat(U, 2, axis=1), np.repeat(F, 2, axis=1)


CH = 64.0


@pytest.mark.parametrize("lim", ["minmod", "mc"])
@pytest.mark.parametrize("axis,sign", [(0, 1), (1, -1), (2, 1), (2, -1)])
@pytest.mark.parametrize("cold", [False, True])
def test_mhd_super_fast_face_has_the_upwind_flux(gd, lim, axis, sign, cold):
    """U' = U - c (F_i - F_{i-1}) with c large, so that the fluxes show. Each flux may
    take two roundings; a cell's sum passes through the transverse flux T that
    stands on both of its sides, which rounds |F_i - F_{i-1}| + |T| twice, and U'
    once; twice that is allowed."""
    U, F = mhd_blocks(sign, cold, seed=23 + axis)
    c, dx = 64.0, 1 / 16
    dF = F - np.roll(F, 1, axis=1) if sign > 0 else np.roll(F, -1, axis=1) - F
    fields = ((1, 2, 3), (5, 6, 7))
    want = U - c * dF
    rho, u, (Bx, By, Bz) = U[0], U[1] / U[0], U[5:8]
    B2, big = Bx * Bx + By * By + Bz * Bz, np.maximum(np.abs(By), np.abs(Bz))
    pT = 0.5 * (U[4] - 0.5 * rho * u * u - 0.5 * B2) + 0.5 * B2
    T = np.stack([0 * u, big * np.abs(Bx), pT + B2, pT + B2, big * np.abs(u * Bx), np.abs(u) * big,
                  0 * u, 0 * u, CH * CH * big])
    off = np.spacing(np.abs(F))
    off += np.roll(off, sign, axis=1)
    tol = 2 * (c * (off + np.spacing(np.abs(dF) + T)) + np.spacing(np.abs(want)))
    say("super-fast faces", lim, axis, sign, "cold" if cold else "warm")
    out = gd.step_mhd(dev(along(rotate(U, axis, fields), axis)), G, dx, c * dx, CH, alpha=0.0,
                      limiter=lim, rho_floor=P_FLOOR, p_floor=P_FLOOR)
    err = np.abs(host(out) - along(rotate(want, axis, fields), axis))
    tol = along(rotate(tol, axis, fields), axis)
    say("worst error in tolerances", float((err / tol).max()))
    assert (err <= tol).all()


def euler_reverse(rho, vel, p, warm, Fb, axis, minus=-1.0):
    """dL/dU of one cell from dL/dF of the flux of its own state along an axis; with
    minus = 1 and all values positive, the sum of the magnitudes of its terms."""
    E = 2.0 * p + 0.5 * rho * (vel @ vel)
    un = vel[axis]
    # F = un (rho, rho vel, E + p) + p e_axis
    Wb = np.zeros((5,) + Fb.shape[1:])
    mom = np.tensordot(vel, Fb[1:4], 1)
    Eb = Fb[4] * un
    Wb[0] = un * (Fb[0] + mom) + Eb * (0.5 * (vel @ vel))
    for d in range(3):
        Wb[1 + d] = rho * un * Fb[1 + d] + Eb * rho * vel[d]
    Wb[1 + axis] += rho * (Fb[0] + mom) + Fb[4] * (E + p)
    Wb[4] = Fb[1 + axis] + Fb[4] * un + 2.0 * Eb
    # p = (U4 - rho vel^2 / 2) / 2, or the floor
    pb = Wb[4] if warm else 0.0 * Wb[4]
    Ub = np.empty_like(Wb)
    Ub[4] = 0.5 * pb
    Ub[0] = Wb[0] + minus * np.tensordot(vel, Wb[1:4], 1) / rho + 0.25 * pb * (vel @ vel)
    for d in range(3):
        Ub[1 + d] = Wb[1 + d] / rho + minus * 0.5 * pb * vel[d]
    return Ub


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("lim", ["minmod", "mc"])
@pytest.mark.parametrize("cold", [False, True])
def test_adjoint_of_supersonic_faces(gd, seed, lim, cold):
    """A uniform state, supersonic along all three axes: dL/dU' comes back through
    the upwind fluxes alone. Each term of a cell's sums passes through fewer than
    sixteen roundings, each at most half a spacing of the sum of magnitudes."""
    rng = np.random.default_rng(seed)
    rho = 2.0 ** rng.integers(-2, 3)
    p = 0.0 if cold else rho * rng.integers(16, 64) / 4.0
    vel = rng.choice([-1, 1], 3) * rng.integers(256, 512, 3) / 8.0
    U = np.array([rho, *(rho * vel), 2.0 * p + 0.5 * rho * (vel @ vel)])
    n = (6, 5, 4)
    lam = rng.integers(-64, 64, (5,) + n) / 8.0
    c, dx = 64.0, 1 / 16
    want, mag = lam.copy(), np.abs(lam)
    for axis in range(3):
        ax = 3 - axis
        step = -1 if vel[axis] > 0 else 1
        # the face downstream of a cell carries its flux
        Fb = c * (np.roll(lam, step, axis=ax) - lam) * (1 if vel[axis] > 0 else -1)
        want += euler_reverse(rho, vel, p, not cold, Fb, axis)
        mag += euler_reverse(rho, np.abs(vel), p, not cold, np.abs(Fb), axis, minus=1.0)
    say("adjoint of supersonic faces", seed, lim, "cold" if cold else "warm")
    got = host(gd.step_adjoint(dev(np.broadcast_to(U.reshape(5, 1, 1, 1), (5,) + n)), dev(lam), G, dx,
                               c * dx, periodic=True, limiter=lim, rho_floor=P_FLOOR,
                               p_floor=P_FLOOR))
    err = np.abs(got - want)
    say("worst error in tolerances", float((err / (8 * np.spacing(mag))).max()))
    assert (err <= 8 * np.spacing(mag)).all()
