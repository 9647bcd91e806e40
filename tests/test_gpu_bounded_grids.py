"""Bounded grids: scal around the edges of a bounded work-group's 8,192
elements, in place and not; bf16, fp8 and binary32 rows whose work-groups are
larger under the bound than without.  Bit for bit."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
import synthetic  # noqa: E402
from oracle import strategies as S  # noqa: E402
from tests.gpu_util import assert_same_bits, to_plan  # noqa: E402
from tests.test_gpu_gemv_codes import check  # noqa: E402


@pytest.mark.parametrize("n", (1025, 8191, 8192, 8193, 8192 * 2 + 4, 8192 * 3 + 1027, 8192 * 5 - 1))
@pytest.mark.parametrize("max_grid", (1, 2, 3))
@pytest.mark.parametrize("in_place", (False, True))
def test_scal(n, max_grid, in_place):
    x = synthetic.normal(synthetic.rng(n), (n + 8,))
    t = torch.from_numpy(x).cuda()
    y = t.clone() if in_place else torch.full_like(t, 7.0)
    s = dp.Strategy(seq_len=64, local_size=256, max_grid=max_grid)
    dp.scal(0.3, y[:n] if in_place else t[:n], s, y=y[:n])
    want = np.concatenate([np.float32(0.3) * x[:n], x[n:] if in_place else np.full(8, 7.0, np.float32)])
    assert_same_bits(y.cpu().numpy(), want, (n, max_grid, in_place))


@pytest.mark.parametrize("dt,L,C,order", ((dp.BF16, 64, 64, dp.STRIDED), (dp.BF16, 512, 19, dp.STRIDED),
                                          (dp.FP8_E4M3, 64, 35, dp.STRIDED), (dp.FP8_E4M3, 256, 11, dp.STRIDED),
                                          (dp.BF16, 128, 64, dp.CONTIGUOUS), (dp.FP8_E4M3, 64, 64, dp.CONTIGUOUS)))
@pytest.mark.parametrize("max_grid", (1, 3, 7))
@pytest.mark.parametrize("combine", (dp.TREE, dp.SEQ))
def test_code_rows(dt, L, C, order, max_grid, combine):
    check(dt, 1203, L * C - 5, dp.Strategy(seq_len=C, local_size=L, order=order, wg_combine=combine,
                                           max_grid=max_grid))


@pytest.mark.parametrize("L,C,order", ((64, 64, dp.STRIDED), (16, 70, dp.STRIDED), (256, 33, dp.STRIDED),
                                       (32, 64, dp.CONTIGUOUS), (16, 128, dp.CONTIGUOUS)))
@pytest.mark.parametrize("max_grid", (1, 3, 300))
def test_binary32_rows(L, C, order, max_grid):
    m, k = 403, L * C - 3
    g = synthetic.rng(k)
    A, x = synthetic.normal(g, (m, k + 3)), synthetic.uniform_pm1(g, k)
    s = dp.Strategy(seq_len=C, local_size=L, order=order, max_grid=max_grid)
    y = dp.gemv(torch.from_numpy(A).cuda()[:, :k], torch.from_numpy(x).cuda(), s)
    assert_same_bits(y.cpu().numpy(), S.gemv(np.ascontiguousarray(A[:, :k]), x, to_plan(s)), (L, C))
