"""GPU parity of FGMRES where its orthogonalization changes kernels: vector
lengths on either side of the one-workgroup form (4,096) and of its lane
counts, odd lengths, and bases of more than 64 vectors (the substitution of the
projections leaves its one-wave form there).  Bars as for the other FGMRES
runs: the oracle's step count, histories to 1e-6, solutions to 1e-7 of their
max norm -- a dot product in another order differs by rounding, which a
history of these well-conditioned systems carries far below that."""
import numpy as np
import pytest

from paper_2111_09512_amd import workloads as W
from tests.gpu_common import assert_close, dev, host, need_gpu, say
from tests.test_gpu_setup_kernels import banded

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    need_gpu()
    from paper_2111_09512_amd import binding

    return binding


@pytest.fixture(scope="module")
def ctx(B):
    return B.Context()


def check(orc, B, ctx, A, restart, m, tol, max_iters, norm_a=None, steps_over=0):
    Ls, U = orc.ilu0(A)
    _, dinv, Us = orc.scale_rows(U)
    F = ctx.ilu_scale_factors(B.Csr.from_host(Ls), B.Csr.from_host(U))
    b, x0 = W.rhs(A.n, 0), W.rhs(A.n, 3) * 0.01
    kw = {} if norm_a is None else {"norm_a": norm_a}
    k_ref, x_ref, h_ref = orc.fgmres(A, Ls, Us, dinv, b, x0, m=restart, max_iters=max_iters, tol=tol, mL=m, mU=m, **kw)
    assert steps_over < k_ref < max_iters
    x = dev(x0)
    k, hist = ctx.fgmres(B.Csr.from_host(A), F, dev(b), x, restart=restart, max_iters=max_iters, tol=tol, m_L=m, m_U=m,
                         **kw)
    assert k == k_ref
    np.testing.assert_allclose(hist, h_ref, rtol=1e-6, atol=1e-15 * h_ref[0])
    assert_close(host(x), x_ref, 1e-7, "fgmres")


@pytest.mark.parametrize("n", [1, 1023, 1025, 2049, 4095, 4096, 4097, 9001])
def test_vector_lengths(orc, B, ctx, n):
    say("arnoldi length", n)
    A = banded(n, 6 if n > 1 else 0, seed=n)
    check(orc, B, ctx, A, 12, 2, 1e-8, 100)


@pytest.mark.parametrize("N", [16, 22])
@pytest.mark.parametrize("norm_a", [None, 12.0])
def test_more_than_64_vectors(orc, B, ctx, N, norm_a):
    say("arnoldi vectors", N, norm_a)
    # one term in either loop: the smoother is a weak preconditioner, and the solve takes more than 64 steps
    check(orc, B, ctx, W.poisson7(N), 120, 1, 1e-9 if norm_a is None else 1e-11, 150, norm_a, steps_over=64)
