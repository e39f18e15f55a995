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


# box, (outer, m_L, m_U), (tile launches, all launches): each form, with a ragged last tile, up to six steps, and a
# reach larger than the tile (23 x 25: tiles of 256 rows)
FORMS = {
    "whole": ((5, 4, 3), (1, 3, 3), (1, 1)),
    "whole_two": ((5, 4, 3), (2, 1, 3), (1, 1)),
    "L_with_residual_and_U": ((16, 16, 17), (1, 5, 5), (2, 2)),
    "L_with_residual_and_U_two": ((30, 9, 40), (2, 3, 4), (4, 4)),
    "L_with_residual_and_U_unequal": ((20, 20, 21), (1, 4, 6), (2, 2)),
    "L_with_residual": ((16, 16, 17), (1, 5, 2), (1, 2)),
    "L_and_U": ((23, 25, 27), (1, 5, 5), (2, 3)),
    "L_and_U_two": ((23, 25, 27), (2, 6, 6), (4, 6)),
    "L_and_U_three_steps": ((32, 33, 31), (1, 3, 3), (2, 3)),
    "L": ((23, 25, 27), (1, 6, 2), (1, 3)),
    "U": ((36, 35, 37), (1, 3, 3), (1, 4)),
    "U_after_one": ((16, 16, 17), (2, 1, 3), (2, 4)),
}


@pytest.mark.parametrize("name", list(FORMS))
def test_forms(orc, B, name):
    from tests.test_gpu_tile import strip

    shape, (outer, m_L, m_U), want = FORMS[name]
    say("tile form", name)
    ctx = B.Context()
    A = strip(*shape)
    Ls, U = orc.ilu0(A)
    d, dinv, Us = orc.scale_rows(U)
    Ad, Ld, Ud = B.Csr.from_host(A), B.Csr.from_host(Ls), B.Csr.from_host(U)
    b, x0 = W.rhs(A.n, 1), W.rhs(A.n, 2)
    bd = dev(b)
    for F in (ctx.ilu_scale_factors(Ld, Ud, fp32=True), ctx.ilu_scale_factors_rowcol(Ld, Ud, 3, fp32=True)):
        for mixed in (False, True):
            for zero in (False, True):
                start = np.zeros(A.n) if zero else x0
                got, plain = dev(start), dev(start)
                seen = launches(ctx, lambda: ctx.ilu_smooth(Ad, F, bd, got, outer, m_L, m_U, mixed=mixed, zero_guess=zero))
                if not mixed and not zero:
                    assert seen == want, seen
                ctx.ilu_smooth(Ad, F, bd, plain, outer, m_L, m_U, mixed=mixed, zero_guess=zero, kernel="rowpat")
                np.testing.assert_array_equal(host(got), host(plain))
                if F.scaled == 1 and not mixed:
                    np.testing.assert_array_equal(host(got), orc.smooth(A, Ls, Us, dinv, b, start, outer, m_L, m_U))
