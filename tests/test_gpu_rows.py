"""Contiguous dots and asums around the lane counts where a launch changes the
lane rows per wavefront (128, 256 and 512 lanes per compute unit), with teams
from 16 lanes to 1,024, row lengths around the tiles (32 to 128 elements),
chunks that share a work-group, and last chunks that end at a row, inside one
and inside a 16-byte part.  Against the oracle, bit for bit."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
import synthetic  # noqa: E402
from oracle import strategies as S  # noqa: E402
from tests.gpu_util import assert_same_bits, to_plan  # noqa: E402


def run(op, n, s, seed):
    g = synthetic.rng(seed)
    x, y = synthetic.uniform_pm1(g, n), synthetic.uniform_pm1(g, n)
    xt, yt = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    code = dp.OP_ASUM if op == "asum" else dp.OP_DOT
    ws = dp.workspace(s, code, dp.F32, 0, n)
    for _ in range(2):                     # the counters are left at zero
        got = (dp.asum(xt, s, ws=ws) if op == "asum" else dp.dot(xt, yt, s, ws=ws)).cpu().numpy()
    want = S.asum(x, to_plan(s)) if op == "asum" else S.dot(x, y, to_plan(s))
    assert_same_bits(np.atleast_1d(got), np.atleast_1d(want), (op, n, s))


@pytest.mark.parametrize("op", ("dot", "asum"))
@pytest.mark.parametrize("L", (16, 32, 64, 128, 256, 512, 1024))
@pytest.mark.parametrize("C", (32, 96, 128, 160, 544))
@pytest.mark.parametrize("end", (0, 1, 2))
def test_rows_and_last_chunks(op, L, C, end):
    combine = (dp.TREE, dp.SEQ)[end == 1]
    s = dp.Strategy(seq_len=C, local_size=L, wg_combine=combine, passes=1 + (end & 1))
    n = 7 * C * L + (0, (L // 2) * C, (L // 3) * C + C // 2 + 3)[end]
    run(op, n, s, L + C)


@pytest.mark.parametrize("op", ("dot", "asum"))
@pytest.mark.parametrize("L,lanes", ((16, 1 << 15), (64, 1 << 15), (32, 1 << 16), (64, 1 << 16)))
@pytest.mark.parametrize("off", (0, 1))
def test_lane_counts(op, L, lanes, off):
    s = dp.Strategy(seq_len=64, local_size=L, passes=1 + off)
    run(op, (lanes // L + off) * 64 * L, s, 3)


@pytest.mark.parametrize("L", (16, 64, 96, 512))
@pytest.mark.parametrize("combine", (dp.TREE, dp.SEQ, dp.NONE))
@pytest.mark.parametrize("C", (8, 40, 72))
def test_vector_lanes(L, combine, C):
    if combine == dp.TREE and L & (L - 1):
        pytest.skip("a tree needs a power of two")
    s = dp.Strategy(seq_len=C, local_size=L, wg_combine=combine, vec_width=4)
    run("dot", 9 * 4 * C * L - 2 * C - 1, s, 5)


@pytest.mark.parametrize("accum", (dp.KAHAN, dp.SUM2))
@pytest.mark.parametrize("L", (16, 64, 256, 1024))
@pytest.mark.parametrize("f64", (0, 1))
def test_compensated(accum, L, f64):
    s = dp.Strategy(seq_len=544, local_size=L, accum=accum, final_f64=f64, passes=1 + f64)
    run("dot", 5 * 544 * L, s, 7)


@pytest.mark.parametrize("max_grid", (1, 3))
def test_bounded_grids(max_grid):
    for L in (16, 64, 512):
        s = dp.Strategy(seq_len=64, local_size=L, max_grid=max_grid, passes=1)
        run("dot", 21 * 64 * L - 5, s, 9)
