"""GPU parity of the row-parallel set-up kernels at the sizes where they can go
wrong: every width of lanes per row, rows longer than that width, rows of one
entry, and row counts on either side of the scan's tiles.  The arithmetic is
the oracle's operation for operation, so every comparison is bit for bit."""
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


@pytest.fixture(scope="module")
def ctx(B):
    return B.Context()


def banded(n, width, long_rows=(), seed=0):
    """Diagonally dominant rows of `width` entries near the diagonal; long_rows couple to every column."""
    rng = np.random.default_rng(seed)
    rows, cols = [np.arange(n)], [np.arange(n)]
    for k in range(1, width // 2 + 1):
        r = np.arange(k, n)
        rows += [r, r - k]
        cols += [r - k, r]
    for r in long_rows:
        c = np.setdiff1d(np.arange(n), np.arange(r - width // 2, r + width // 2 + 1))
        rows.append(np.full(c.size, r))
        cols.append(c)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    vals = -rng.uniform(0.1, 1.0, rows.size)
    on = rows == cols
    vals[on] = 0.0
    tot = np.zeros(n)
    np.add.at(tot, rows, -vals)
    np.add.at(tot, cols, -vals)
    vals[on] = tot + 0.5
    return W._coo_to_csr(n, rows, cols, vals)


# (rows, entries near the diagonal, rows that couple to every column)
SHAPES = [(1, 0, ()), (2, 2, ()), (3000, 4, (5,)), (257, 6, (3, 250)), (2048, 8, ()), (2049, 14, (0, 2048)), (700, 15, ()),
          (700, 30, (350,)), (4100, 34, (4099,)), (300, 62, ()), (300, 90, (7, 8, 299))]


@pytest.mark.parametrize("n,width,long_rows", SHAPES)
def test_fixed_point_rows_of_every_width(orc, B, ctx, n, width, long_rows):
    say("fixed point", n, width, long_rows)
    A = banded(n, width, long_rows, seed=n + width)
    for sweeps in (1, 3):
        Ls, U, _ = orc.ilu0_fixed_point(A, sweeps)
        gL, gU, _ = ctx.ilu0_fixed_point(B.Csr.from_host(A), sweeps)
        for g, ref in ((gL, Ls), (gU, U)):
            np.testing.assert_array_equal(host(g.row_ptr), ref.row_ptr)
            np.testing.assert_array_equal(host(g.col_idx), ref.col)
            np.testing.assert_array_equal(host(g.val), ref.val)


@pytest.mark.parametrize("n,width,long_rows", SHAPES)
def test_gauss_seidel_split_rows_of_every_width(orc, B, ctx, n, width, long_rows):
    say("gs split", n, width, long_rows)
    A = banded(n, width, long_rows, seed=n + width)
    Gs, dinv = orc.gs_split(A)
    G = ctx.gs_split(B.Csr.from_host(A), fp32=True)
    np.testing.assert_array_equal(host(G.Ls.row_ptr), Gs.row_ptr)
    np.testing.assert_array_equal(host(G.Ls.col_idx), Gs.col)
    np.testing.assert_array_equal(host(G.Ls.val), Gs.val)
    np.testing.assert_array_equal(host(G.d), A.val[A.col == np.repeat(np.arange(n), np.diff(A.row_ptr))])
    np.testing.assert_array_equal(host(G.dinv), dinv)
    np.testing.assert_array_equal(host(G.Ls_val32), Gs.val.astype(np.float32))


@pytest.mark.parametrize("scale", [True, False])
@pytest.mark.parametrize("n,width,long_rows", SHAPES + [(256, 4, ()), (513, 40, (0, 255, 256))])
def test_scale_factors_rows_of_every_width(orc, B, ctx, n, width, long_rows, scale):
    say("scale", n, width, long_rows, scale)
    A = banded(n, width, long_rows, seed=n + width)
    Ls, U = orc.ilu0(A)
    d, dinv, Us = orc.scale_rows(U)
    if not scale:
        Us.val[:] = U.val[U.col != np.repeat(np.arange(n), np.diff(U.row_ptr))]
    F = ctx.ilu_scale_factors(B.Csr.from_host(Ls), B.Csr.from_host(U), fp32=True, scale=scale)
    np.testing.assert_array_equal(host(F.Us.row_ptr), Us.row_ptr)
    np.testing.assert_array_equal(host(F.Us.col_idx), Us.col)
    np.testing.assert_array_equal(host(F.Us.val), Us.val)
    np.testing.assert_array_equal(host(F.Us_val32), Us.val.astype(np.float32))
    np.testing.assert_array_equal(host(F.Ls_val32), Ls.val.astype(np.float32))
    np.testing.assert_array_equal(host(F.d), d)
    np.testing.assert_array_equal(host(F.dinv), dinv)
