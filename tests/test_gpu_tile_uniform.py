"""A face between two tiles is solved by both, and a cell beside it is predicted by
both: by its own tile, and by the other one's ring. Data that vary along one axis
only show whether the two do the same arithmetic: the same bits in every cell
across that axis, on a box of several tiles, z-ranges and remainders."""
import numpy as np
import pytest

from helpers import say
from paper_1412_0934_amd import inputs

pytestmark = pytest.mark.gpu
G = 5.0 / 3.0
N = (60, 40, 20)


@pytest.fixture(scope="module")
def gd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1412_0934_amd import godunov
    return godunov


def along(line, axis, fields):
    """Data [var][i] along x turned to an axis, as a box [var][z][y][x] of N cells."""
    import torch
    v = np.array(line)
    for f in fields:
        v[[f[(c + axis) % 3] for c in range(3)]] = line[list(f)]
    one = [1, 1, 1]
    one[2 - axis] = N[axis]
    u = np.broadcast_to(v.reshape([len(v)] + one), (len(v),) + N[::-1])
    return torch.from_numpy(np.ascontiguousarray(u)).to("cuda")


def assert_uniform(t, axis):
    import torch
    torch.cuda.synchronize()
    out = t.cpu().numpy()
    row = tuple(slice(None) if d in (0, 3 - axis) else slice(0, 1) for d in range(4))
    assert np.array_equal(out, np.broadcast_to(out[row], out.shape))


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("rs", ["hllc", "hll"])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_step(gd, axis, rs, dtype):
    import torch
    line = inputs.random_patch(N[axis], 1, 1, ng=2, seed=3 + axis, generic=True)[:, 2, 2, 2:-2]
    u = along(line, axis, ((1, 2, 3),)).to(getattr(torch, dtype))
    for lim in ("minmod", "mc", "none", "ppm", "ppm_unlimited", "ppm_ct", "ppm_ct_unlimited"):
        say("transverse-uniform", axis, rs, dtype, lim)
        out, _ = gd.step(u, G, 1 / 64, 1e-3, periodic=True, limiter=lim, riemann=rs)
        assert_uniform(out, axis)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("lim", ["minmod", "mc", "none"])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_mhd_step(gd, axis, lim, dtype):
    import torch
    line = inputs.mhd_random_box(N[axis], 1, 1, seed=40 + axis)[:, 0, 0, :]
    u = along(line, axis, ((1, 2, 3), (5, 6, 7))).to(getattr(torch, dtype))
    say("mhd transverse-uniform", axis, lim, dtype)
    assert_uniform(gd.step_mhd(u, G, 1 / 64, 1e-3, 3.0, alpha=0.1, limiter=lim), axis)
