"""The adjoint differentiates the branch that the forward step took, also where
rounding decides it. On a pressure that rises linearly, each minmod slope is the
smaller of two differences that are equal but for the rounding of the primitive
conversion. That rounding is reproduced here exactly, in rational arithmetic, in
the order of the step's conversion (fused multiply-adds; density one, so that its
reciprocal is exact); then the pressure is bent by 1e-7 a cell towards the same
branches, which decides them beyond rounding. The two adjoints agree up to the
bend, 1e-7 n^2 / 2 of the pressure; a single branch taken otherwise changes them by
order one."""
from fractions import Fraction

import numpy as np
import pytest

import oracle
from helpers import say

pytestmark = pytest.mark.gpu
G = 5.0 / 3.0
N = 20


@pytest.fixture(scope="module")
def gd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1412_0934_amd import godunov
    return godunov


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def pressure(U):
    return (G - 1.0) * fma(-0.5, fma(U[3], U[3], fma(U[2], U[2], U[1] * U[1])), U[4])


@pytest.mark.parametrize("seed", range(8))
@pytest.mark.parametrize("riemann", ["hllc", "hll"])
@pytest.mark.parametrize("axis", [0, 2])
def test_limiter_branches_at_rounding(gd, seed, riemann, axis):
    import torch
    rng = np.random.default_rng(seed)
    m = N + 4
    vel = rng.standard_normal((3, m))

    # the velocity turned with the axis: the conversion sums its components in order
    turn = [0, *(1 + (c - axis) % 3 for c in range(3)), 4]

    def state(p):
        return np.stack([np.ones(m), *vel, p / (G - 1.0) + 0.5 * (vel ** 2).sum(axis=0)])

    rise = 1.0 + 0.05 * np.arange(m)
    U = state(rise)
    d = np.diff([pressure([float(x) for x in U[turn, i]]) for i in range(m)])
    bend = np.zeros(m)
    for i in range(1, m - 1):
        lower = abs(d[i - 1]) <= abs(d[i])
        bend[i + 1] = 2 * bend[i] - bend[i - 1] + (1e-7 if lower else -1e-7)
    lam = rng.standard_normal((5, N))

    def adjoint(U):
        one, cells, inside = [1, 1, 1], [6, 6, 6], [2, 2, 2]
        one[2 - axis], cells[2 - axis], inside[2 - axis] = -1, m, N
        one_lam = [N if c == -1 else c for c in one]
        u = np.broadcast_to(U[turn].reshape([5] + one), [5] + cells)
        lo = np.broadcast_to(lam[turn].reshape([5] + one_lam), [5] + inside)
        t = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (u, lo)]
        out = gd.step_adjoint(t[0], t[1], G, 1 / 64, 2e-3, limiter="minmod", riemann=riemann)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    say("adjoint branches at rounding", seed, riemann, axis)
    off = np.abs(adjoint(U) - adjoint(state(rise + bend))).max()
    say("largest difference", float(off))
    assert off <= 1e-3


@pytest.mark.parametrize("shape", [(50, 20, 9), (25, 9, 33), (2, 30, 17)])
@pytest.mark.parametrize("limiter,riemann", [("minmod", "hllc"), ("mc", "hll"), ("none", "hllc")])
def test_smooth_periodic_boxes_that_are_no_cubes(gd, shape, limiter, riemann):
    """Against the oracle to 1e-12, as everywhere: smooth waves of generic phase, whose
    limiter branches rounding does not decide."""
    import torch
    nx, ny, nz = shape
    rng = np.random.default_rng(nx)
    z, y, x = np.meshgrid(*((np.arange(n) + 0.5) / n for n in (nz, ny, nx)), indexing="ij")

    def wave(base, amplitude):
        f = np.full(x.shape, base)
        for _ in range(3):
            k, phase = rng.integers(-2, 3, 3), rng.uniform(0, 2 * np.pi)
            f += amplitude * np.sin(2 * np.pi * (k[0] * x + k[1] * y + k[2] * z) + phase)
        return f

    rho, p, v = wave(1.0, 0.1), wave(1.0, 0.1), [wave(0.2, 0.2) for _ in range(3)]
    u = np.stack([rho, *(rho * c for c in v), p / (G - 1.0) + 0.5 * rho * sum(c * c for c in v)])
    lam = rng.standard_normal(u.shape)
    lb = rng.standard_normal(oracle.bflux_size(nx, ny, nz))
    dx = 1 / 64
    dt = 0.5 * oracle.cfl_dt(u, G, dx, periodic=True)
    want = oracle.step_adjoint(u, lam, G, dx, dt, lam_bflux=lb, limiter=limiter, riemann=riemann,
                               periodic=True)
    say("smooth periodic adjoint", shape, limiter, riemann)
    got = gd.step_adjoint(*(torch.from_numpy(a).cuda() for a in (u, lam)), G, dx, dt,
                          lam_bflux=torch.from_numpy(lb).cuda(), limiter=limiter, riemann=riemann,
                          periodic=True)
    torch.cuda.synchronize()
    assert float(np.abs(got.cpu().numpy() - want).max() / np.abs(want).max()) <= 1e-12
