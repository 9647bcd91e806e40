"""Strided dots and asums around the lane counts where a launch changes from 4
lanes per thread to one (256 or 512 lanes per compute unit), with chunks of
one wavefront and of several, lengths that leave partial chunks and
remainders of every batch size, and 1-pass launches around the 256 work-groups
beyond which their arrivals are counted in two levels.  Against the oracle,
bit for bit."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
import synthetic  # noqa: E402
from oracle import strategies as S  # noqa: E402
from tests.gpu_util import assert_same_bits, to_plan  # noqa: E402

CUS = 256


def run(op, n, s, seed):
    g = synthetic.rng(seed)
    x, y = synthetic.uniform_pm1(g, n), synthetic.uniform_pm1(g, n)
    if op == "i32":
        x, y = (synthetic.integers_u32(g, n).view(np.int32) for _ in range(2))
    xt, yt = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    ws = dp.workspace(s, dp.OP_ASUM if op == "asum" else dp.OP_DOT,
                      dp.I32 if op == "i32" else dp.F32, 0, n)
    for _ in range(2):                     # the counters are left at zero
        got = (dp.asum(xt, s, ws=ws) if op == "asum" else dp.dot(xt, yt, s, ws=ws)).cpu().numpy()
    if op == "asum":
        want = S.asum(x, to_plan(s))
    elif op == "i32":
        got, want = got.view(np.uint32), S.dot(x.view(np.uint32), y.view(np.uint32), to_plan(s), num="u32")
    else:
        want = S.dot(x, y, to_plan(s))
    assert_same_bits(np.atleast_1d(got), np.atleast_1d(want), (op, n, s))


# lanes in the launch below, at and above each change, by lanes per chunk
@pytest.mark.parametrize("op,limit", (("dot", 256 * CUS), ("asum", 512 * CUS), ("i32", 256 * CUS)))
@pytest.mark.parametrize("L", (16, 64, 256, 512, 1024))
@pytest.mark.parametrize("off", (-1, 0, 1))
@pytest.mark.parametrize("combine", (dp.TREE, dp.SEQ))
def test_lane_counts(op, limit, L, off, combine):
    s = dp.Strategy(seq_len=5, local_size=L, order=dp.STRIDED, wg_combine=combine,
                    passes=1 + (off & 1))
    chunks = limit // L + off
    run(op, (chunks - 1) * 5 * L + 3 * L + 7, s, 3)


# few chunks: remainders of a 64-step batch of every size
@pytest.mark.parametrize("op", ("dot", "asum", "i32"))
@pytest.mark.parametrize("C", (1, 63, 64, 65, 95, 127, 161))
@pytest.mark.parametrize("L", (4, 48, 64, 512))
def test_batch_remainders(op, C, L):
    tree = L & (L - 1) == 0
    s = dp.Strategy(seq_len=C, local_size=L, order=dp.STRIDED,
                    wg_combine=dp.TREE if tree else dp.SEQ, passes=1)
    run(op, 3 * C * L + (C // 2) * L + 1, s, 5)


@pytest.mark.parametrize("accum", (dp.KAHAN, dp.SUM2))
@pytest.mark.parametrize("C,L", ((77, 64), (130, 16), (9, 1024)))
def test_compensated(accum, C, L):
    s = dp.Strategy(seq_len=C, local_size=L, order=dp.STRIDED, accum=accum, passes=1)
    run("dot", 5 * C * L, s, 7)


@pytest.mark.parametrize("groups", (255, 256, 257, 289, 512, 1001))
@pytest.mark.parametrize("order", (dp.STRIDED, dp.CONTIGUOUS))
def test_arrivals(groups, order):
    # one chunk per work-group of 256 threads (1,024 strided lanes)
    L = 1024 if order == dp.STRIDED else 256
    s = dp.Strategy(seq_len=32, local_size=L, order=order, passes=1)
    run("dot", groups * 32 * L, s, 9)
