"""GPU parity of the smoother on matrices small enough that several sweeps
share a launch: sizes on either side of one workgroup's, one to many tiles with
a ragged last one, every count of inner steps on either side, both precisions,
the zero guess, repeated outer steps and both scalings, against the oracle (FP64
bit for bit) and against the same call on the row-pattern copies, which always
takes a launch per sweep (bit for bit in both precisions)."""
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
def ctx(B):
    return B.Context()


def strip(nx, ny, nz):
    """7-point operator on an nx x ny x nz box: its reach is nx ny, its size nx ny nz."""
    n = nx * ny * nz
    i = np.arange(n)
    x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
    rng = np.random.default_rng(n)
    rows, cols, vals = [i], [i], [6.5 + rng.random(n)]
    for ok, step in ((x > 0, -1), (x < nx - 1, 1), (y > 0, -nx), (y < ny - 1, nx), (z > 0, -nx * ny),
                     (z < nz - 1, nx * ny)):
        rows.append(i[ok])
        cols.append(i[ok] + step)
        vals.append(-rng.uniform(0.5, 1.0, ok.sum()))
    return W._coo_to_csr(n, np.concatenate(rows), np.concatenate(cols), np.concatenate(vals))


SHAPES = {"one_row_wide": (2, 1, 1), "small": (5, 4, 3), "coarse": (16, 16, 16), "whole_edge": (16, 16, 26),
          "past_whole": (16, 16, 27), "thin": (7, 5, 700), "tiles": (20, 20, 41), "side31": (31, 31, 31),
          "flat": (3000, 2, 3), "long_reach": (64, 64, 9)}


@pytest.fixture(scope="module")
def cases(orc, B, ctx):
    out = {}
    for name, shape in SHAPES.items():
        A = strip(*shape)
        Ls, U = orc.ilu0(A)
        d, dinv, Us = orc.scale_rows(U)
        Ld, Ud = B.Csr.from_host(Ls), B.Csr.from_host(U)
        out[name] = dict(A=A, Ls=Ls, Us=Us, dinv=dinv, Ad=B.Csr.from_host(A), F=ctx.ilu_scale_factors(Ld, Ud, fp32=True),
                         Frc=ctx.ilu_scale_factors_rowcol(Ld, Ud, 3, fp32=True), Ld=Ld, Ud=Ud)
    return out


@pytest.mark.parametrize("steps", [(1, 1, 1), (1, 2, 2), (1, 3, 3), (2, 3, 3), (1, 4, 4), (3, 5, 2), (1, 2, 6), (2, 1, 3),
                                   (2, 3, 1), (1, 6, 6)])
@pytest.mark.parametrize("name", list(SHAPES))
def test_tiles_equal_sweeps(orc, ctx, cases, name, steps):
    say("tile", name, steps)
    c = cases[name]
    n = c["A"].n
    outer, m_L, m_U = steps
    b, x0 = W.rhs(n, 1), W.rhs(n, 2)
    bd = dev(b)
    ref = orc.smooth(c["A"], c["Ls"], c["Us"], c["dinv"], b, x0, outer, m_L, m_U)
    for F in (c["F"], c["Frc"]):
        for mixed in (False, True):
            for zero in (False, True):
                start = np.zeros(n) if zero else x0
                got, plain = dev(start), dev(start)
                ctx.ilu_smooth(c["Ad"], F, bd, got, outer, m_L, m_U, mixed=mixed, zero_guess=zero)
                ctx.ilu_smooth(c["Ad"], F, bd, plain, outer, m_L, m_U, mixed=mixed, zero_guess=zero, kernel="rowpat")
                np.testing.assert_array_equal(host(got), host(plain))
                if F is c["F"] and not mixed and not zero:
                    np.testing.assert_array_equal(host(got), ref)


def test_replays_and_runs_in_a_row(ctx, cases):
    """A recorded call and calls one after the other on one workspace, nothing waited for between them."""
    say("tile replays")
    for name in ("coarse", "tiles"):
        c = cases[name]
        n = c["A"].n
        bd = dev(W.rhs(n, 3))
        ws = ctx.workspace(n)
        want = torch.zeros_like(bd)
        for _ in range(4):
            ctx.ilu_smooth(c["Ad"], c["F"], bd, want, 1, 3, 3, kernel="rowpat")
        got, rec = torch.zeros_like(bd), torch.zeros_like(bd)
        for _ in range(4):
            ctx.ilu_smooth(c["Ad"], c["F"], bd, got, 1, 3, 3, ws=ws)
            ctx.ilu_smooth(c["Ad"], c["F"], bd, rec, 1, 3, 3, ws=ws, record=True)
        np.testing.assert_array_equal(host(got), host(want))
        np.testing.assert_array_equal(host(rec), host(want))
