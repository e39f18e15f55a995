"""The context makes a sliced copy of a matrix only when a sweep of the call
reads it: none of a factor with one inner step, none of A where the only
residual is that of a declared zero guess.  Shown by values changed where the
context is not told: a copy made too early would still hold the old ones."""
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


@pytest.mark.parametrize("op", ["poisson", "perm"])
@pytest.mark.parametrize("mixed", [False, True])
def test_copies_follow_the_sweeps(orc, B, op, mixed):
    say("copies", op, mixed)
    A = W.poisson7(20) if op == "poisson" else W.permuted_longrange7(20, seed=1)
    Ls, U = orc.ilu0(A)
    ctx = B.Context()
    b = dev(W.rhs(A.n, 1))

    def device():
        """A and its factors, in arrays of their own."""
        return B.Csr.from_host(A), ctx.ilu_scale_factors(B.Csr.from_host(Ls), B.Csr.from_host(U), fp32=True)

    def halve(*tensors):
        for t in tensors:
            t.data.mul_(0.5)  # leaves the version counter, so the binding releases nothing

    def call(Ad, F, m_L, m_U, zero=False):
        x = torch.zeros_like(b)
        ctx.ilu_smooth(Ad, F, b, x, 1, m_L, m_U, mixed=mixed, zero_guess=zero)
        return host(x)

    def want(halved, m_L, m_U, zero=False):
        Ad, F = device()
        halve(*halved(Ad, F))
        return call(Ad, F, m_L, m_U, zero)

    def lower(Ad, F):
        return F.Ls.val, F.Ls_val32

    def upper(Ad, F):
        return F.Us.val, F.Us_val32

    Ad, F = device()
    call(Ad, F, 1, 1)
    halve(*lower(Ad, F), *upper(Ad, F))
    np.testing.assert_array_equal(call(Ad, F, 3, 3), want(lambda *s: lower(*s) + upper(*s), 3, 3))
    Ad, F = device()
    call(Ad, F, 2, 1)
    halve(*upper(Ad, F))
    np.testing.assert_array_equal(call(Ad, F, 2, 2), want(upper, 2, 2))
    Ad, F = device()
    call(Ad, F, 1, 2)
    halve(*lower(Ad, F))
    np.testing.assert_array_equal(call(Ad, F, 2, 2), want(lower, 2, 2))
    Ad, F = device()
    call(Ad, F, 2, 2, zero=True)
    halve(Ad.val)
    np.testing.assert_array_equal(call(Ad, F, 2, 2), want(lambda Ad, F: (Ad.val,), 2, 2))
