"""GPU parity of the level-scheduled substitution where its launches change
form: levels on either side of the width that one workgroup takes, runs of
levels cut where a row reaches further back than the on-chip window, rows of
more entries than a lane holds, rows shared by 64 lanes, and long chains of
one-row levels; lower and upper, unit and stored diagonals.  Bar: 1e-12 of the
solution's maximum, as for the other substitutions (bit for bit where a row is
summed in storage order by one lane)."""
import numpy as np
import pytest
import torch

from paper_2111_09512_amd import workloads as W
from tests.gpu_common import F64_TOL, assert_close, dev, host, need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    need_gpu()
    from paper_2111_09512_amd import binding

    return binding


@pytest.fixture(scope="module")
def ctx(B):
    return B.Context()


def lower(widths, deps, seed):
    """A strictly lower triangle with levels of the given widths: every row of a level couples to a row of the
    level before it and to the rows that deps(rng, level, first row of the level) picks among the earlier ones."""
    rng = np.random.default_rng(seed)
    rows, cols, start = [], [], 0
    for lv, w in enumerate(widths):
        if lv:
            prev = start - widths[lv - 1]
            for r in range(start, start + w):
                c = np.unique(np.append(deps(rng, lv, start), rng.integers(prev, start)))
                rows.append(np.full(c.size, r))
                cols.append(c)
        start += w
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    length = np.bincount(rows, minlength=start)
    vals = rng.uniform(-1.0, 1.0, rows.size) / np.maximum(length, 1)[rows]  # row sums below 1: no growth
    return W._coo_to_csr(start, rows, cols, vals)


def few(k):
    return lambda rng, lv, s: rng.integers(0, s, k)


CASES = {
    # one-row levels
    "chain": lambda: lower([1] * 3000, lambda rng, lv, s: rng.integers(max(0, s - 3), s, 1), 1),
    # 500 levels of 90 rows that reach back 30,000 rows: past the window (16,384)
    "far": lambda: lower([90] * 500, lambda rng, lv, s: np.maximum(0, s - 1 - rng.integers(0, 30000, 2)), 2),
    # just within the window
    "near": lambda: lower([90] * 300, lambda rng, lv, s: np.maximum(0, s - 1 - rng.integers(0, 16384 - 180, 2)), 3),
    # narrow, wide, narrow levels
    "wide": lambda: lower([500, 16000, 9000, 65, 64, 63, 1] + [40] * 40 + [20000, 7, 300, 14000] + [33] * 30, few(3), 4),
    # rows of 21 to 60 entries (more than a lane holds)
    "rows60": lambda: lower([200] * 60, lambda rng, lv, s: rng.integers(0, s, rng.integers(20, 60)), 5),
    # single rows of hundreds and thousands of entries among short ones
    "long": lambda: lower([18000, 70, 1, 130, 2, 64] + [20] * 50, lambda rng, lv, s: rng.integers(
        0, s, rng.choice([2, 3, 250, 257, 2500], p=[0.45, 0.45, 0.04, 0.03, 0.03])), 6),
    # too few levels for the layout: a launch each
    "shallow": lambda: lower([700, 500, 64, 1, 900], few(4), 7),
}
EXACT = ("chain", "near", "rows60")  # summed in storage order: nothing is read from before the window


@pytest.mark.parametrize("name", list(CASES))
def test_substitution(orc, B, ctx, name):
    say("levels", name)
    T = CASES[name]()
    n = T.n
    rhs = W.rhs(n, 1)
    rows = np.repeat(np.arange(n), np.diff(T.row_ptr))
    every = np.arange(n)
    diag = np.random.default_rng(7).uniform(1.0, 2.0, n)
    with_diag = W._coo_to_csr(n, np.append(rows, every), np.append(T.col, every), np.append(T.val, diag))
    # the mirror image: row n - 1 - i, an upper triangle with the same levels
    flip = W._coo_to_csr(n, n - 1 - rows, n - 1 - T.col.astype(np.int64), T.val)
    flip_diag = W._coo_to_csr(n, np.append(n - 1 - rows, every), np.append(n - 1 - T.col.astype(np.int64), every),
                              np.append(T.val, diag))
    for M, uplo, unit in ((T, "L", True), (with_diag, "L", False), (flip, "U", True), (flip_diag, "U", False)):
        ref = orc.trisolve(M, uplo, unit, rhs)
        Md = B.Csr.from_host(M)
        out = None
        for rep in range(2):
            got = host(ctx.trisolve_direct(Md, B.SILU_LOWER if uplo == "L" else B.SILU_UPPER,
                                           B.SILU_UNIT if unit else B.SILU_NONUNIT, dev(rhs)))
            assert_close(got, ref, F64_TOL, f"{name} {uplo} unit={unit}")
            if out is not None:
                np.testing.assert_array_equal(got, out)
            out = got
        if name in EXACT:
            np.testing.assert_array_equal(out, ref)


def test_values_changed_in_place_are_read(orc, B, ctx):
    """The layout holds the pattern only: a solve reads the values as they are."""
    say("levels, new values")
    T = CASES["rows60"]()
    Td = B.Csr.from_host(T)
    rhs = W.rhs(T.n, 2)
    out = dev(np.zeros(T.n))

    def solve():  # past the binding, which would release the analysis
        import ctypes as C

        Tc = Td.c()
        assert B._lib.trisolve_direct(ctx._h, C.byref(Tc), B.SILU_LOWER, B.SILU_UNIT, C.c_void_p(rd.data_ptr()),
                                      C.c_void_p(out.data_ptr()), 0) == 0
        return host(out)

    rd = dev(rhs)
    assert_close(solve(), orc.trisolve(T, "L", True, rhs), F64_TOL, "values")
    Td.val.mul_(0.5)
    T.val[:] = 0.5 * T.val
    assert_close(solve(), orc.trisolve(T, "L", True, rhs), F64_TOL, "values")


def test_two_streams_share_a_layout(orc, B, ctx):
    """Solves of one context on two streams in turn, nothing waited for between them."""
    say("levels, two streams")
    T = CASES["far"]()
    Td = B.Csr.from_host(T)
    rhs = [dev(W.rhs(T.n, 10 + k)) for k in range(6)]
    out = [torch.empty_like(r) for r in rhs]
    ref = [orc.trisolve(T, "L", True, host(r)) for r in rhs]
    side = torch.cuda.Stream()
    ctx.trisolve_direct(Td, B.SILU_LOWER, B.SILU_UNIT, rhs[0], out[0])
    torch.cuda.synchronize()
    try:
        for k in range(6):
            s = side if k & 1 else ctx.stream
            B._lib.silu_set_stream(ctx._h, s.cuda_stream)
            ctx.trisolve_direct(Td, B.SILU_LOWER, B.SILU_UNIT, rhs[k], out[k])
    finally:
        B._lib.silu_set_stream(ctx._h, ctx.stream.cuda_stream)
    torch.cuda.synchronize()
    for o, r in zip(out, ref):
        assert_close(host(o), r, F64_TOL, "two streams")


def test_nonfinite_values_stay_with_their_rows(orc, B, ctx):
    """An infinite right-hand side entry reaches the rows that depend on it, and no others."""
    say("levels, infinity")
    for name in ("far", "wide", "long"):
        T = CASES[name]()
        rhs = W.rhs(T.n, 4)
        rhs[T.n // 2] = np.inf
        with np.errstate(all="ignore"):
            ref = orc.trisolve(T, "L", True, rhs)
        got = host(ctx.trisolve_direct(B.Csr.from_host(T), B.SILU_LOWER, B.SILU_UNIT, dev(rhs)))
        np.testing.assert_array_equal(np.isfinite(got), np.isfinite(ref))
        assert 0 < np.isfinite(ref).sum() < T.n
        fin = np.isfinite(ref)
        assert_close(got[fin], ref[fin], F64_TOL, name)
