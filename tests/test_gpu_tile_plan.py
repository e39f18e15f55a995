"""Which calls on small matrices take several sweeps a launch: not those whose
sweeps by themselves keep the device far shorter (one workgroup for a whole call
on 16^3 points), and in a recording, which costs the host one launch whatever it
holds, none that keep it longer at all.  Results are the same either way."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2111_09512_amd import workloads as W
from tests.gpu_common import dev, host, need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    need_gpu()
    from paper_2111_09512_amd import binding

    return binding


@pytest.fixture(scope="module")
def hip(B):
    """The HIP runtime that the process has loaded."""
    with open("/proc/self/maps") as f:
        paths = {ln.split()[-1] for ln in f if "libamdhip64" in ln}
    assert len(paths) == 1, paths
    return C.CDLL(paths.pop())


def case(B, ctx, N):
    A = W.poisson7(N)
    L, U = B.factor_iluk(A, 0)
    return B.Csr.from_host(A), ctx.ilu_scale_factors(B.Csr.from_host(L), B.Csr.from_host(U)), dev(W.rhs(A.n, 1))


def launches(ctx, call):
    """Launches of an eager call: (those of tile kernels, all)."""
    ctx.set_timing(True)
    ctx.stats_reset()
    call()
    st = ctx.stats()
    ctx.set_timing(False)
    return st.get("smooth_tile", {"launches": 0})["launches"], sum(v["launches"] for v in st.values())


def recorded(B, ctx, hip, call):
    """(kernel nodes, executable graph) of the call captured on a stream of its own."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    s, g, ex, n = C.c_void_p(side.cuda_stream), C.c_void_p(), C.c_void_p(), C.c_size_t()
    B._lib.silu_set_stream(ctx._h, side.cuda_stream)
    try:
        assert hip.hipStreamBeginCapture(s, 1) == 0  # thread-local
        call()
        assert hip.hipStreamEndCapture(s, C.byref(g)) == 0
    finally:
        B._lib.silu_set_stream(ctx._h, ctx.stream.cuda_stream)
    assert hip.hipGraphGetNodes(g, None, C.byref(n)) == 0
    assert hip.hipGraphInstantiate(C.byref(ex), g, None, None, C.c_size_t(0)) == 0
    return n.value, g, ex


@pytest.mark.parametrize("N,steps,tiles", [(10, (1, 3), True), (16, (1, 1), False), (14, (1, 1), False), (16, (1, 3), True),
                                           (16, (2, 4), True), (48, (1, 3), False)])
def test_eager_plans(B, N, steps, tiles):
    say("tile plan", N, steps)
    ctx = B.Context()
    Ad, F, b = case(B, ctx, N)
    x, plain = torch.zeros_like(b), torch.zeros_like(b)
    tiled, every = launches(ctx, lambda: ctx.ilu_smooth(Ad, F, b, x, steps[0], steps[1]))
    assert (tiled > 0) == tiles, (tiled, every)
    ctx.ilu_smooth(Ad, F, b, plain, steps[0], steps[1], kernel="rowpat")
    np.testing.assert_array_equal(host(x), host(plain))


@pytest.mark.parametrize("N,steps,nodes", [(24, (4, 3), 20), (32, (2, 4), 14), (10, (4, 3), 1)])
def test_recorded_plans(B, hip, N, steps, nodes):
    say("tile plan recorded", N, steps)
    ctx = B.Context()
    Ad, F, b = case(B, ctx, N)
    x, plain = torch.zeros_like(b), torch.zeros_like(b)
    ws = ctx.workspace(b.numel())

    def call():
        ctx.ilu_smooth(Ad, F, b, x, steps[0], steps[1], ws=ws)

    assert launches(ctx, call)[0] > 0  # in tiles where it is not recorded
    torch.cuda.synchronize()
    n, g, ex = recorded(B, ctx, hip, call)
    assert n == nodes
    ctx.ilu_smooth(Ad, F, b, plain, steps[0], steps[1], kernel="rowpat")
    want = host(plain)
    for rep in range(3):
        x.zero_()
        assert hip.hipGraphLaunch(ex, C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        np.testing.assert_array_equal(host(x), want)
        junk = torch.randn(4096, device="cuda").cumsum(0)
        torch.cuda.synchronize()
        assert torch.isfinite(junk).all()
    assert hip.hipGraphExecDestroy(ex) == 0 and hip.hipGraphDestroy(g) == 0
