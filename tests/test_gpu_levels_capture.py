"""Direct solves recorded into the caller's own graph: recordable right after
the level analysis (nothing is allocated or waited for in the capture), and
replayed beside eager solves with the same triangle on another stream, nothing
waited for between them.  Bar: 1e-12 of the solution's maximum, as for the other
substitutions."""
import numpy as np
import pytest
import torch

from paper_2111_09512_amd import workloads as W
from tests.gpu_common import F64_TOL, assert_close, dev, host, need_gpu, say
from tests.test_gpu_levels import CASES

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    need_gpu()
    from paper_2111_09512_amd import binding

    return binding


def capture(B, ctx, call):
    """call() recorded on a stream of its own."""
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    B._lib.silu_set_stream(ctx._h, side.cuda_stream)
    try:
        with torch.cuda.graph(g, stream=side):
            call()
    finally:
        B._lib.silu_set_stream(ctx._h, ctx.stream.cuda_stream)
    return g


@pytest.mark.parametrize("name", ["far", "wide", "long", "shallow"])
def test_recorded_solve_beside_eager_ones(orc, B, name):
    say("levels captured", name)
    ctx = B.Context()
    T = CASES[name]()
    Td = B.Csr.from_host(T)
    rhs = [W.rhs(T.n, 30 + k) for k in range(8)]
    ref = [orc.trisolve(T, "L", True, r) for r in rhs]
    rd = [dev(r) for r in rhs]
    rec_rhs, rec_out = dev(rhs[0]), torch.zeros(T.n, dtype=torch.float64, device="cuda")
    out = [torch.zeros_like(r) for r in rd]
    ctx.silu_analyze(Td, B.SILU_LOWER)
    torch.cuda.synchronize()
    ctx.set_timing(True)
    ctx.trisolve_direct(Td, B.SILU_LOWER, B.SILU_UNIT, rd[0], out[0])
    copied = any(k.startswith("level_pack") for k in ctx.stats())
    ctx.set_timing(False)
    assert copied == (name != "shallow")  # "shallow" has no level-ordered copy
    # a context that has solved nothing yet records its first solve
    fresh = B.Context()
    fresh.silu_analyze(Td, B.SILU_LOWER)
    graph = capture(B, fresh, lambda: fresh.trisolve_direct(Td, B.SILU_LOWER, B.SILU_UNIT, rec_rhs, rec_out))
    shared = capture(B, ctx, lambda: ctx.trisolve_direct(Td, B.SILU_LOWER, B.SILU_UNIT, rec_rhs, rec_out))
    for g in (graph, shared):
        for rep in range(3):
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            replayed = []
            for k in range(0, 8, 2):
                with torch.cuda.stream(side):
                    rec_rhs.copy_(rd[k])
                    g.replay()
                    replayed.append(rec_out.clone())
                ctx.trisolve_direct(Td, B.SILU_LOWER, B.SILU_UNIT, rd[k + 1], out[k + 1])
            torch.cuda.synchronize()
            for k in range(0, 8, 2):
                assert_close(host(replayed[k // 2]), ref[k], F64_TOL, f"{name} replay {rep}")
                assert_close(host(out[k + 1]), ref[k + 1], F64_TOL, f"{name} eager {rep}")


def test_recorded_direct_smoother(orc, B):
    say("direct smoother captured")
    ctx = B.Context()
    A = W.vardens7(13)
    Ls, U = orc.iluk(A, 1)
    d, dinv, Us = orc.scale_rows(U)
    Ad, F = B.Csr.from_host(A), ctx.ilu_scale_factors(B.Csr.from_host(Ls), B.Csr.from_host(U))
    b, x0 = W.rhs(A.n, 1), W.rhs(A.n, 2)
    ref = orc.smooth(A, Ls, Us, dinv, b, x0, 1, 0, 0, direct=True)
    bd, x = dev(b), dev(x0)
    ctx.ilu_smooth(Ad, F, bd, x, 1, 1, 1, direct=True)  # the residual's layout is made here
    eager = host(x)
    assert_close(eager, ref, F64_TOL, "eager")
    g = capture(B, ctx, lambda: ctx.ilu_smooth(Ad, F, bd, x, 1, 1, 1, direct=True))
    for rep in range(4):
        x.copy_(dev(x0))
        torch.cuda.synchronize()
        g.replay()
        assert_close(host(x), ref, F64_TOL, f"replay {rep}")
        junk = torch.randn(4096, device="cuda").cumsum(0)
        torch.cuda.synchronize()
        assert torch.isfinite(junk).all()
        x.copy_(dev(x0))
        ctx.ilu_smooth(Ad, F, bd, x, 1, 1, 1, direct=True)
        np.testing.assert_array_equal(host(x), eager)
