"""Strided chunks fed by loader wavefronts whose last one is only partly there:
one wavefront folds that alone, in batches of 64 steps, so its steps end
before, at and after such a batch.  Against the oracle, bit for bit."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
from tests.test_gpu_thin import run  # noqa: E402


@pytest.mark.parametrize("op", ("dot", "asum"))
@pytest.mark.parametrize("L", (16, 64, 256))
@pytest.mark.parametrize("steps", (0, 1, 63, 64, 65, 128, 1023))
def test_steps_of_the_last_chunk(op, L, steps):
    s = dp.Strategy(seq_len=1024, local_size=L, order=dp.STRIDED, wg_combine=dp.TREE)
    run(op, 3 * 1024 * L + steps * L + L // 2 + 1, s, 5)
