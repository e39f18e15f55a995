"""GPU tests of batched serving sweeps that share a matrix between requests:
steps large enough that requests on one matrix are swept in groups (a group of
more, of as many and of fewer ops than the loads are batched by), on copies of
one and two groups of slots, on wider rows, on a ragged last slice and beside
matrices that are not shared.  Each request equals the same request run alone
bit for bit."""
import numpy as np
import pytest
import torch

from paper_2111_09512_amd import workloads as W
from tests.gpu_common import dev, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    need_gpu()
    from paper_2111_09512_amd import binding

    return binding


@pytest.fixture(scope="module")
def ctx(B):
    return B.Context()


@pytest.fixture(scope="module")
def pool(orc, B, ctx):
    mats = [W.vardens7(41, seed_rho=3, with_cuts=False), W.vardens7(40, seed_rho=4, with_cuts=True), W.aniso27(19),
            W.vardens7(9, seed_rho=5, with_cuts=False)]
    out = []
    for k, A in enumerate(mats):
        L, U = B.factor_iluk(A, 0)
        Ad, Ld, Ud = B.Csr.from_host(A), B.Csr.from_host(L), B.Csr.from_host(U)
        F = ctx.ilu_scale_factors_rowcol(Ld, Ud, 3, fp32=True) if k == 1 else ctx.ilu_scale_factors(Ld, Ud, fp32=True)
        out.append((A.n, Ad, F, Ud))
    torch.cuda.synchronize()
    return out


# requests on each matrix; the first has 270 workgroups a sweep, so 12 and more of them are swept in groups
@pytest.mark.parametrize("counts", [(12, 0, 0, 0), (13, 0, 4, 3), (30, 9, 5, 2), (9, 30, 0, 1)])
@pytest.mark.parametrize("mixed", [False, True])
def test_requests_on_shared_matrices_equal_the_single_call(B, ctx, pool, counts, mixed):
    server = B.Server(ctx, arena_bytes=1 << 30)
    mids = [server.register(Ad, F) for _, Ad, F, _ in pool]
    rng = np.random.default_rng(sum(counts))
    which = rng.permutation(np.repeat(np.arange(4), counts))
    reqs = []
    for k, j in enumerate(which):
        n = pool[j][0]
        mL, mU = [(3, 3), (2, 4), (1, 3), (4, 1), (3, 3), (3, 3)][k % 6]
        reqs.append((j, dev(W.rhs(n, 100 + k)), dev(W.rhs(n, 500 + k) * (k % 2)), 1 + k % 2, mL, mU))
    alone = []
    for j, b, x, outer, mL, mU in reqs:
        _, Ad, F, _ = pool[j]
        y = x.clone()
        ctx.ilu_smooth(Ad, F, b, y, outer, mL, mU, mixed=mixed)
        alone.append(host(y))
    for j, b, x, outer, mL, mU in reqs:
        server.submit(mids[j], b, x, outer, mL, mU, mixed=mixed)
    for _ in range(1000):
        active, queued = server.run(8)
        if not active and not queued:
            break
    torch.cuda.synchronize()
    for (j, _, x, *_), want in zip(reqs, alone):
        assert np.array_equal(host(x), want), f"matrix {j}"


def test_solve_requests_on_a_shared_matrix(B, ctx, pool):
    """Solve requests (whose check ops stay by themselves and whose stopped
    sweeps are skipped) beside smoothing requests on the same matrix."""
    n, Ad, F, _ = pool[0]

    def run(server, count):
        mid = server.register(Ad, F)
        xs, tickets = [], []
        for k in range(count):
            x = dev(np.zeros(n))
            b = dev(W.rhs(n, 900 + k))
            xs.append((b, x))
            tickets.append(server.submit_solve(mid, b, x, [0.3, 1e-2, 1e-3][k % 3], 6, 3, 3) if k % 2 else
                           server.submit(mid, b, x, 3, 3, 3))
        for _ in range(1000):
            active, queued = server.run(8)
            if not active and not queued:
                break
        torch.cuda.synchronize()
        server.completed()
        return [host(x) for _, x in xs], [server.solve_result(t) for t in tickets[1::2]]

    got, res = run(B.Server(ctx, arena_bytes=1 << 30), 26)
    for k in range(0, 26, 5): # by themselves: a server that has nothing to share
        alone = B.Server(ctx, arena_bytes=1 << 30)
        mid = alone.register(Ad, F)
        x, b = dev(np.zeros(n)), dev(W.rhs(n, 900 + k))
        t = alone.submit_solve(mid, b, x, [0.3, 1e-2, 1e-3][k % 3], 6, 3, 3) if k % 2 else alone.submit(mid, b, x, 3, 3, 3)
        for _ in range(1000):
            active, queued = alone.run(8)
            if not active and not queued:
                break
        torch.cuda.synchronize()
        alone.completed()
        assert np.array_equal(host(x), got[k])
        if k % 2:
            assert alone.solve_result(t) == res[k // 2]
