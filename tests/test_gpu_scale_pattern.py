"""Row scaling of a U whose row pointers do not ascend or leave its arrays: an
error naming a row, from the kernel's own checks (no entry outside the arrays is
read), where a block of 256 rows begins, inside one and at the end."""
import numpy as np
import pytest

from paper_2111_09512_amd import workloads as W
from tests.gpu_common import host, need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    need_gpu()
    from paper_2111_09512_amd import binding

    return binding


@pytest.mark.parametrize("at", [256, 300, 512, 600])
@pytest.mark.parametrize("value", [-1, -(1 << 30), "behind", 1 << 30, (1 << 31) - 1])
def test_row_pointers_outside_the_arrays(orc, B, at, value):
    say("scale pattern", at, value)
    ctx = B.Context()
    A = W.poisson7(9)
    Ls, U = orc.ilu0(A)
    n, nnz = 600, int(U.row_ptr[600])
    rp = U.row_ptr[: n + 1].copy()
    keep = U.col[:nnz] < n
    col, val = U.col[:nnz][keep], U.val[:nnz][keep]  # the leading 600 rows and columns
    rows = np.repeat(np.arange(n), np.diff(rp))[keep]
    good = W._coo_to_csr(n, rows, col, val)
    low = np.repeat(np.arange(n), np.diff(Ls.row_ptr[: n + 1]))
    lower = W._coo_to_csr(n, low, Ls.col[: low.size], Ls.val[: low.size])
    F = ctx.ilu_scale_factors(B.Csr.from_host(lower), B.Csr.from_host(good), fp32=True)
    d, dinv, Us = orc.scale_rows(good)
    np.testing.assert_array_equal(host(F.Us.val), Us.val)
    bad = W.CSR(n, good.row_ptr.copy(), good.col, good.val)
    bad.row_ptr[at] = good.col.size + 1 if value == "behind" else value
    with pytest.raises(B.SiluError) as e:
        ctx.ilu_scale_factors(B.Csr.from_host(lower), B.Csr.from_host(bad), fp32=True)
    assert B.STATUS[e.value.status] == "SILU_ERR_PATTERN"
    assert at - 1 <= e.value.row <= at


# U's entries on either side of the line between the two kernels, and rows that one lane does not take by itself
@pytest.mark.parametrize("n,width", [(4, 1), (255, 64), (257, 65), (1000, 66), (2500, 200), (174762, 3), (174763, 3),
                                     (131072, 4), (131073, 4), (400000, 4)])
@pytest.mark.parametrize("dense_first", [False, True])
@pytest.mark.parametrize("scale", [True, False])
def test_both_forms(B, n, width, dense_first, scale):
    say("scale forms", n, width, dense_first, scale)
    rng = np.random.default_rng(n + width)
    length = np.minimum(width, n - np.arange(n))
    if dense_first:  # one row of every column, up to 3,000
        length[0] = min(n, 3000)
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(length, out=rp[1:])
    row = np.repeat(np.arange(n), length)
    first = np.arange(rp[-1]) - rp[row]
    U = W.CSR(n, rp.astype(np.int32), (row + first).astype(np.int32), rng.uniform(0.5, 2.0, rp[-1]))
    L = W.CSR(n, np.concatenate([[0], np.arange(n)]).astype(np.int32), np.arange(n - 1, dtype=np.int32),
              rng.uniform(0.5, 2.0, n - 1))
    off = first > 0
    piv = U.val[~off]
    F = B.Context().ilu_scale_factors(B.Csr.from_host(L), B.Csr.from_host(U), fp32=True, scale=scale)
    val = U.val[off] / piv[row[off]] if scale else U.val[off]
    np.testing.assert_array_equal(host(F.Us.row_ptr), rp - np.arange(n + 1))
    np.testing.assert_array_equal(host(F.Us.col_idx), U.col[off])
    np.testing.assert_array_equal(host(F.Us.val), val)
    np.testing.assert_array_equal(host(F.Us_val32), val.astype(np.float32))
    np.testing.assert_array_equal(host(F.d), piv)
    np.testing.assert_array_equal(host(F.dinv), 1.0 / piv)
