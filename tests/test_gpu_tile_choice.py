"""The library's own choice of tiles is a setting of its own: reported as such,
distinct from every fixed configuration, and the initial one. On boxes of several
24x8 tiles it runs those, in z-ranges of several planes, and gives the bits of 16x16
tiles (the kernels that ran are read from a trace)."""
import ctypes

import numpy as np
import pytest

from helpers import say
from paper_1412_0934_amd import inputs

pytestmark = pytest.mark.gpu
G = 5.0 / 3.0


@pytest.fixture(scope="module")
def gd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1412_0934_amd import godunov
    return godunov


def traced(f):
    """f()'s result and the names of the step kernels it launched."""
    import torch
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        out = f()
        torch.cuda.synchronize()
    return out, [e.key for e in p.key_averages() if "step_" in e.key and "kernel" in e.key]


def test_a_setting_of_its_own(gd):
    import torch
    ctx = gd.Context(torch.cuda.current_device())
    v = [ctypes.c_int(7) for _ in range(4)]

    def config():
        ctx.check(ctx.lib.gd_get_config(ctx.handle, 0, *[ctypes.byref(x) for x in v]))
        return [x.value for x in v]

    assert config()[0] == -1 and config()[2] == -1
    assert ctx.lib.gd_set_config(ctx.handle, 0, 0, 32, 0, 1) == 0 and config() == [0, 32, 0, 1]
    assert ctx.lib.gd_set_config(ctx.handle, 0, -2, 32, 0, 1) != 0
    assert ctx.lib.gd_set_config(ctx.handle, 0, 0, 32, -2, 1) != 0
    assert config() == [0, 32, 0, 1]
    assert ctx.lib.gd_set_config(ctx.handle, 0, -1, 32, -1, 1) == 0
    assert config()[0] == -1 and config()[2] == -1

    f64 = torch.float64
    fixed = dict(shape_single="16x16", zlen_single=32, shape_batched="16x16", zpolicy_batched=1)
    try:
        gd.set_config(f64)
        own = gd.get_config(f64)
        assert own["shape_single"] == own["shape_batched"] == "auto"
        gd.set_config(f64, **fixed)
        assert gd.get_config(f64) == fixed
        gd.set_config(f64, zlen_single=16, zpolicy_batched=2)
        assert gd.get_config(f64) == dict(fixed, zlen_single=16, zpolicy_batched=2)
        gd.set_config(f64, **own)
        assert gd.get_config(f64) == own
        say("autotune from the library's own choice")
        u = torch.from_numpy(inputs.random_patch(40, 24, 16, seed=1)).cuda()
        choice = gd.autotune_step(u, G, 1 / 64, 1e-3)
        tuned = gd.get_config(f64)
        order = ("16x16", "32x8", "8x8", "16x8", "24x8")
        assert tuned["shape_single"] in ("auto", order[choice // 3])
        assert tuned["shape_single"] == "auto" or tuned["zlen_single"] == (16, 32, 64)[choice % 3]
    finally:
        gd.set_config(f64)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("lim,rs", [("minmod", "hllc"), ("mc", "hll")])
@pytest.mark.parametrize("shape,periodic", [((192, 128, 30), True), ((168, 72, 40), False)])
def test_single_patches_of_several_tiles(gd, dtype, lim, rs, shape, periodic):
    import torch
    dt_ = getattr(torch, dtype)
    u = inputs.random_patch(*shape, ng=0 if periodic else 2, seed=5, generic=True)
    d = torch.from_numpy(u).cuda().to(dt_)

    def step():
        return gd.step(d, G, 1 / 64, 1e-3, periodic=periodic, limiter=lim, riemann=rs)

    say("own tiles", dtype, lim, rs, shape)
    own, ran = traced(step)
    assert len(ran) == 1 and ", 24, 8>" in ran[0]
    try:
        gd.set_config(dt_, shape_single="16x16", zlen_single=32)
        fixed, ran = traced(step)
        assert len(ran) == 1 and ", 16, 16>" in ran[0]
    finally:
        gd.set_config(dt_)
    for a, b in zip(own, fixed):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_batches(gd, dtype):
    import torch
    dt_ = getattr(torch, dtype)
    rng = np.random.default_rng(8)
    states = [inputs.random_patch(*(int(v) for v in rng.integers(4, 30, size=3)), seed=400 + p,
                                  generic=True) for p in range(40)]
    batch = inputs.pack_batch(states, 2, 1 / 64, order_seed=6)
    table = gd.patch_table(batch.dims, 2, batch.u_in_off, batch.u_out_off, batch.flux_off,
                           batch.dx, 1e-3)
    u_in = torch.from_numpy(batch.u_in).cuda().to(dt_)

    def step():
        out = torch.zeros(batch.u_out_size, dtype=dt_, device="cuda")
        flux = torch.zeros(batch.flux_size, dtype=dt_, device="cuda")
        gd.step_batched(u_in, table, G, out=out, bflux=flux)
        return out, flux

    say("own tiles of a batch", dtype)
    own, ran = traced(step)
    assert len(ran) == 1 and ", 24, 8>" in ran[0]       # 24x8 alone or the pair
    try:
        gd.set_config(dt_, shape_batched="16x16", zpolicy_batched=1)
        fixed, ran = traced(step)
        assert len(ran) == 1 and ", 16, 16>" in ran[0]
    finally:
        gd.set_config(dt_)
    for a, b in zip(own, fixed):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,npatch,n", [("float32", 64, 32), ("float64", 256, 16)])
def test_batches_of_patches_that_fill_16x16_tiles(gd, dtype, npatch, n):
    """Alike patches whose 16x16 tiles find one place each on the chip: those are
    chosen (by 20 to 25% the fastest), and give the bits of the tile pair."""
    import torch
    dt_ = getattr(torch, dtype)
    states = [inputs.random_patch(n, n, n, seed=q, generic=True) for q in range(4)]
    batch = inputs.pack_batch([states[p % 4] for p in range(npatch)], 2, 1 / 64, order_seed=2)
    table = gd.patch_table(batch.dims, 2, batch.u_in_off, batch.u_out_off, batch.flux_off,
                           batch.dx, 1e-3)
    u_in = torch.from_numpy(batch.u_in).cuda().to(dt_)

    def step():
        out = torch.zeros(batch.u_out_size, dtype=dt_, device="cuda")
        flux = torch.zeros(batch.flux_size, dtype=dt_, device="cuda")
        gd.step_batched(u_in, table, G, out=out, bflux=flux)
        return out, flux

    say("alike patches", dtype, npatch, n)
    own, ran = traced(step)
    assert len(ran) == 1 and ", 16, 16>" in ran[0]
    try:
        gd.set_config(dt_, shape_batched="16x8+24x8", zpolicy_batched=2)
        pair, ran = traced(step)
        assert len(ran) == 1 and "pair" in ran[0]
    finally:
        gd.set_config(dt_)
    for a, b in zip(own, pair):
        assert torch.equal(a, b)
