"""FGMRES above 4,096 rows where orthogonalization is hard: a basis that is
exhausted (the preconditioned operator has five distinct eigenvalues), iterating
on at the accuracy limit across restarts (the new directions nearly depend on the
old), and stalling restarts.  The projections come there from products with the
vector as it was (a triangular system that is modified Gram-Schmidt's recurrence),
so their rounding differs from one projection at a time; it is of the same order.
Bars: the true residual, summed in extended precision, within four times that of
the oracle's modified Gram-Schmidt plus four units of rounding; where the history
is far from rounding, the oracle's history to 1e-6 and its step count."""
import numpy as np
import pytest

from paper_2111_09512_amd import workloads as W
from tests.gpu_common import dev, host, need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    need_gpu()
    from paper_2111_09512_amd import binding

    return binding


def diagonal(d):
    """Rows of one coupling that is 0, and the diagonal d."""
    n, i = d.size, np.arange(d.size)
    return W._coo_to_csr(n, np.append(i, i[1:]), np.append(i, i[:-1]), np.append(d, np.zeros(n - 1)))


def relres(A, b, x):
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    ax = np.zeros(A.n, np.longdouble)
    np.add.at(ax, rows, A.val.astype(np.longdouble) * x.astype(np.longdouble)[A.col])
    return float(np.sqrt(np.sum((b - ax) ** 2)) / np.linalg.norm(b))


def solve(orc, B, A, Ls, U, b, restart, max_iters, tol, m):
    _, dinv, Us = orc.scale_rows(U)
    k_ref, x_ref, h_ref = orc.fgmres(A, Ls, Us, dinv, b, np.zeros(A.n), m=restart, max_iters=max_iters, tol=tol, mL=m, mU=m)
    ctx = B.Context()
    F = ctx.ilu_scale_factors(B.Csr.from_host(Ls), B.Csr.from_host(U))
    x = dev(np.zeros(A.n))
    k, h = ctx.fgmres(B.Csr.from_host(A), F, dev(b), x, restart=restart, max_iters=max_iters, tol=tol, m_L=m, m_U=m)
    got, ref = relres(A, b, host(x)), relres(A, b, x_ref)
    print("steps", k, k_ref, "residual", got, ref, flush=True)
    return k, k_ref, h, h_ref, got, ref


EPS = np.finfo(float).eps


@pytest.mark.parametrize("n", [4097, 6000, 20011])
def test_exhausted_basis(orc, B, n):
    say("arnoldi exhausted", n)
    A = diagonal(np.array([1.0, 2.0, 5.0, 11.0, 30.0])[np.arange(n) % 5])
    i = np.arange(n)
    Ls = W._coo_to_csr(n, i[1:], i[:-1], np.zeros(n - 1))
    U = W._coo_to_csr(n, i, i, np.ones(n))  # M = I
    *_, got, ref = solve(orc, B, A, Ls, U, W.rhs(n, 2), 12, 24, 0.0, 1)
    assert got <= 4 * ref + 4 * EPS


@pytest.mark.parametrize("N,restart,max_iters", [(18, 100, 150), (20, 60, 90), (22, 30, 90)])
def test_beyond_the_accuracy_limit(orc, B, N, restart, max_iters):
    say("arnoldi limit", N, restart)
    A = W.poisson7(N)
    Ls, U = orc.ilu0(A)
    *_, got, ref = solve(orc, B, A, Ls, U, W.rhs(A.n, 1), restart, max_iters, 0.0, 3)
    assert got <= 4 * ref + 4 * EPS


@pytest.mark.parametrize("restart", [5, 10, 40])
def test_stalling_restarts(orc, B, restart):
    """An upwind chain without a preconditioner: the residual falls like a power of the step count."""
    say("arnoldi stall", restart)
    n = 6000
    i = np.arange(n)
    A = W._coo_to_csr(n, np.append(i, i[1:]), np.append(i, i[:-1]), np.append(np.ones(n), -np.ones(n - 1)))
    Ls = W._coo_to_csr(n, i[1:], i[:-1], -np.ones(n - 1))
    U = W._coo_to_csr(n, i, i, np.ones(n))
    b = np.zeros(n)
    b[0] = 1.0
    k, k_ref, h, h_ref, got, ref = solve(orc, B, A, Ls, U, b, restart, 120, 1e-10, 1)
    assert k == k_ref == 120
    np.testing.assert_allclose(h, h_ref, rtol=1e-6)
    assert abs(got - ref) <= 1e-6 * ref


def test_no_direction_behind_the_last_step(B):
    """A solve that stops after its first step applies the preconditioner once."""
    say("arnoldi one step")
    A = W.poisson7(20)
    L, U = B.factor_iluk(A, 0)
    ctx = B.Context()
    F = ctx.ilu_scale_factors(B.Csr.from_host(L), B.Csr.from_host(U))
    Ad, b, x = B.Csr.from_host(A), dev(W.rhs(A.n, 1)), dev(np.zeros(A.n))
    ctx.set_timing(True)
    k, _ = ctx.fgmres(Ad, F, b, x, restart=30, max_iters=60, tol=0.5, m_L=3, m_U=3, kernel="rowpat")
    sweeps = sum(v["launches"] for name, v in ctx.stats().items() if name.startswith("sweep"))
    assert k == 1
    assert sweeps == 1 + 4 + 1  # the first residual, one smoother call from zero, the product with A
