"""Direct solves that take a launch per level: a sequence that comes again with
the same arrays is replayed from a graph, which changes no bit; sequences that
come once are not captured, however many there are."""
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


def launches(ctx, call):
    ctx.set_timing(True)
    ctx.stats_reset()
    call()
    st = {k: v["launches"] for k, v in ctx.stats().items() if v["launches"]}
    ctx.set_timing(False)
    return st


def test_repeated_solves_replay(orc, B):
    say("level graph")
    ctx = B.Context()
    T = CASES["shallow"]()
    Td = B.Csr.from_host(T)
    depth, _ = ctx.silu_analyze(Td, B.SILU_LOWER)
    rd, out = dev(W.rhs(T.n, 1)), torch.zeros(T.n, dtype=torch.float64, device="cuda")

    def solve(graph=True):
        ctx.trisolve_direct(Td, B.SILU_LOWER, B.SILU_UNIT, rd, out, graph=graph)

    assert launches(ctx, solve) == {"level_f64": depth}  # seen once
    for rep in range(4):
        rhs = W.rhs(T.n, 10 + rep)
        rd.copy_(dev(rhs))
        assert launches(ctx, solve) == {"level_graph": 1}
        got = host(out)
        assert_close(got, orc.trisolve(T, "L", True, rhs), F64_TOL, f"replay {rep}")
        junk = torch.randn(4096, device="cuda").cumsum(0)
        torch.cuda.synchronize()
        assert torch.isfinite(junk).all()
        out.zero_()
        assert launches(ctx, lambda: solve(False)) == {"level_f64": depth}
        np.testing.assert_array_equal(host(out), got)
    # other arrays: their own sequence; many of them once each leave room for one that comes again
    outs = [torch.zeros_like(out) for _ in range(80)]
    for o in outs:
        ctx.trisolve_direct(Td, B.SILU_LOWER, B.SILU_UNIT, rd, o)
    want = host(out)
    for o in outs:
        np.testing.assert_array_equal(host(o), want)
    outs[-1].zero_()
    last = launches(ctx, lambda: ctx.trisolve_direct(Td, B.SILU_LOWER, B.SILU_UNIT, rd, outs[-1]))
    assert last == {"level_graph": 1}
    np.testing.assert_array_equal(host(outs[-1]), want)
    # values changed in place: the analysis is made again, and so is the sequence
    Td.val.mul_(0.5)
    T.val[:] = 0.5 * T.val
    for rep in range(3):
        solve()
        assert_close(host(out), orc.trisolve(T, "L", True, host(rd)), F64_TOL, f"new values {rep}")


def test_direct_smoother_on_few_levels(orc, B):
    """The smoother on a randomly permuted operator, whose factors have a few wide levels."""
    say("level graph, smoother")
    ctx = B.Context()
    A = W.permuted_longrange7(24, seed=1)
    Ls, U = orc.ilu0(A)
    d, dinv, Us = orc.scale_rows(U)
    Ad, F = B.Csr.from_host(A), ctx.ilu_scale_factors(B.Csr.from_host(Ls), B.Csr.from_host(U))
    b, x0 = W.rhs(A.n, 1), W.rhs(A.n, 2)
    ref = orc.smooth(A, Ls, Us, dinv, b, x0, 1, 0, 0, direct=True)
    bd, x = dev(b), dev(x0)
    first = None
    for rep in range(4):
        x.copy_(dev(x0))
        ctx.ilu_smooth(Ad, F, bd, x, 1, 1, 1, direct=True, graph=rep != 3)
        got = host(x)
        assert_close(got, ref, F64_TOL, f"call {rep}")
        first = got if first is None else first
        if rep < 3:
            np.testing.assert_array_equal(got, first)
