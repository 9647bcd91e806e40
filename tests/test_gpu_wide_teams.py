"""Strided dots and asums whose lanes need teams of more than 256 threads (no
four of them to a thread), with few chunks and load batches of every
remainder.  Against the oracle, bit for bit."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
from tests.test_gpu_thin import run  # noqa: E402


@pytest.mark.parametrize("op", ("dot", "asum", "i32"))
@pytest.mark.parametrize("C", (1, 7, 16, 33, 79))
@pytest.mark.parametrize("L", (257, 514, 1022))
def test_batch_remainders(op, C, L):
    s = dp.Strategy(seq_len=C, local_size=L, order=dp.STRIDED, wg_combine=dp.SEQ, passes=1)
    run(op, 3 * C * L + (C // 2) * L + 1, s, 5)


@pytest.mark.parametrize("accum", (dp.KAHAN, dp.SUM2))
@pytest.mark.parametrize("L", (257, 514, 1022))
def test_compensated(accum, L):
    s = dp.Strategy(seq_len=79, local_size=L, order=dp.STRIDED, wg_combine=dp.SEQ, accum=accum,
                    passes=1)
    run("dot", 5 * 79 * L, s, 7)
