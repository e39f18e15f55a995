"""Level-scheduled substitution at the edge of the on-chip window: a row that
reads the oldest solution still held there stays in its run of levels, one that
reads the position before it starts a new run, after what it reads further back
was subtracted.  Rows are then summed in storage order either way (all of such a
row's entries lie before its run), so results are the oracle's bit for bit."""
import re
from pathlib import Path

import numpy as np
import pytest

from paper_2111_09512_amd import workloads as W
from tests.gpu_common import dev, host, need_gpu, say

pytestmark = pytest.mark.gpu

SOURCE = Path(__file__).resolve().parents[1] / "paper_2111_09512_amd" / "csrc" / "internal.h"
RING = int(re.search(r"LEVEL_RING = (\d+);", SOURCE.read_text()).group(1))
WIDTH, LEVELS = 90, 300


@pytest.fixture(scope="module")
def B():
    need_gpu()
    from paper_2111_09512_amd import binding

    return binding


def ladder(level, back, mirrored):
    """A strictly lower triangle of LEVELS levels of WIDTH rows, each row coupled to one row of the level before;
    the rows of `level` also to the one at position `back` before the level's end.  Positions number the rows level
    by level and by index in a level: in the mirror image a level's rows are the other way round."""
    rng = np.random.default_rng(3)
    n = WIDTH * LEVELS
    rows = np.arange(WIDTH, n)
    cols = (rows // WIDTH - 1) * WIDTH + rng.integers(0, WIDTH, rows.size)
    extra, at = np.arange(level * WIDTH, (level + 1) * WIDTH), (level + 1) * WIDTH - back
    if mirrored:
        at = at // WIDTH * WIDTH + WIDTH - 1 - at % WIDTH
    rows, cols = np.append(rows, extra), np.append(cols, np.full(WIDTH, at))
    return W._coo_to_csr(n, rows, cols, rng.uniform(-0.5, 0.5, rows.size))


@pytest.mark.parametrize("uplo", ["L", "U"])
@pytest.mark.parametrize("level", [227, 250, 280])
@pytest.mark.parametrize("past,runs,far", [(0, 1, 0), (1, 2, 1)])
def test_edge_of_the_window(orc, B, uplo, level, past, runs, far):
    say("levels ring", uplo, level, past)
    assert 228 * WIDTH > RING  # level 227 can read past the window
    T = ladder(level, RING + past, uplo == "U")
    n = T.n
    if uplo == "U":  # the mirror image: an upper triangle with the same levels
        rows = np.repeat(np.arange(n), np.diff(T.row_ptr))
        T = W._coo_to_csr(n, n - 1 - rows, n - 1 - T.col.astype(np.int64), T.val)
    rhs = W.rhs(n, 1)
    ctx = B.Context()
    ctx.set_timing(True)
    got = host(ctx.trisolve_direct(B.Csr.from_host(T), B.SILU_LOWER if uplo == "L" else B.SILU_UPPER, B.SILU_UNIT,
                                   dev(rhs)))
    st = ctx.stats()
    np.testing.assert_array_equal(got, orc.trisolve(T, uplo, True, rhs))
    count = {k: st.get(k, {"launches": 0})["launches"] for k in ("level_run", "level_far", "level_wide")}
    assert count == {"level_run": runs, "level_far": far, "level_wide": 0}, count
