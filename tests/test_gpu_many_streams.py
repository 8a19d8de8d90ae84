"""More streams than a context has counter slots: reductions that overlap on a
shared slot may spoil each other's time step (they are documented to interfere),
but no later one's."""
import ctypes

import numpy as np
import pytest

import oracle
from helpers import say
from paper_1412_0934_amd import inputs

pytestmark = pytest.mark.gpu
G = 5.0 / 3.0
STREAMS, SLOTS = 70, 64


@pytest.fixture(scope="module")
def gd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1412_0934_amd import godunov
    return godunov


def test_reductions_on_shared_slots(gd):
    import torch
    ctx = gd.Context(torch.cuda.current_device())
    hip = ctx.lib               # finds the HIP runtime that the library is linked with
    streams = [ctypes.c_void_p() for _ in range(STREAMS)]
    for s in streams:
        assert hip.hipStreamCreate(ctypes.byref(s)) == 0
    opts = gd.gd_opts(0, 0, 0, 0, 1e-10, 1e-10)
    # grids of different size: 2, 41 and 128 workgroups
    sizes = [(8, 8, 8), (24, 20, 22), (32, 32, 32)]
    states = [inputs.random_patch(*s, seed=p, generic=True) for p, s in enumerate(sizes)]
    want = [oracle.cfl_dt(u, G, 1 / 64, 0.5) for u in states]
    dev = [torch.from_numpy(u).cuda() for u in states]
    out = torch.full((STREAMS,), -1.0, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()

    def reduce(i, k):
        desc = gd.gd_patch(*sizes[k], 2, 0, 0, -1, 1 / 64, 0.0)
        ctx.check(ctx.lib.cfl_dt(ctx.handle, ctypes.byref(opts), 1, ctypes.addressof(desc),
                                 dev[k].data_ptr(), G, 0.5, out[i].data_ptr(), streams[i].value))

    try:
        for i in range(STREAMS):                # every stream has its slot
            reduce(i, 0)
            torch.cuda.synchronize()
        say("overlapping reductions on shared slots")
        for _ in range(20):
            for i in range(SLOTS, STREAMS):
                reduce(i, i % 3)
                reduce(i - SLOTS, (i + 1) % 3)
        torch.cuda.synchronize()
        for i in list(range(SLOTS, STREAMS)) + list(range(STREAMS - SLOTS)):
            for k in range(3):
                say("one at a time", i, k)
                out.fill_(-1.0)
                torch.cuda.synchronize()
                reduce(i, k)
                torch.cuda.synchronize()
                got = float(out[i].cpu())
                assert abs(got - want[k]) <= 1e-14 * want[k]
    finally:
        torch.cuda.synchronize()
        for s in streams:
            hip.hipStreamDestroy(s)
