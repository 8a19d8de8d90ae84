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
