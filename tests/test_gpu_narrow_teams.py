"""1-pass launches of many chunks of a few strided lanes, on both sides of where
the lanes are one to a thread.  Against the oracle, bit for bit."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
from tests.test_gpu_thin import run  # noqa: E402


@pytest.mark.parametrize("op", ("dot", "asum", "i32"))
@pytest.mark.parametrize("L,lanes", ((4, 16384), (8, 16384), (16, 32768), (32, 49152)))
@pytest.mark.parametrize("C", (1, 7, 18))
def test_lines(op, L, lanes, C):
    s = dp.Strategy(seq_len=C, local_size=L, order=dp.STRIDED, wg_combine=dp.TREE, passes=1)
    for n in ((lanes - L) * C, lanes * C, lanes * C - 1, (lanes - L) * C + 1):
        run(op, n, s, 5)


@pytest.mark.parametrize("accum", (dp.KAHAN, dp.SUM2))
@pytest.mark.parametrize("L,lanes", ((4, 16384), (16, 32768), (32, 49152)))
def test_compensated(accum, L, lanes):
    s = dp.Strategy(seq_len=7, local_size=L, order=dp.STRIDED, wg_combine=dp.TREE, passes=1,
                    accum=accum)
    run("dot", lanes * 7, s, 7)
