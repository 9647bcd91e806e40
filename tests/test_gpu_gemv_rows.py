"""bf16 and fp8 gemv rows under the strided order, at the row counts where the
launch changes between 4, 2 and 1 rows per team and between load batches, with
row lengths that leave remainders of every size, a part of a last step, and
rows past a work-group's last.  Against the oracle, bit for bit."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
import synthetic  # noqa: E402
from oracle import strategies as S  # noqa: E402
from tests.gpu_util import assert_same_bits, to_plan  # noqa: E402


def rows_of(m):
    """The rows compared: all of a small matrix, else both ends and some between."""
    if m <= 600:
        return np.arange(m)
    return np.unique(np.concatenate([np.arange(64), np.arange(m - 64, m),
                                     np.random.default_rng(m).integers(0, m, 200)]))


def check(kind, m, k, s, lda):
    g = synthetic.rng(m + k)
    A, x = synthetic.normal(g, (m, lda)), synthetic.uniform_pm1(g, k)
    at = rows_of(m)
    xt = torch.from_numpy(x).cuda()
    if kind == "bf16":
        codes = synthetic.quantise_bf16(A)
        y = dp.gemv(torch.from_numpy(codes.view(np.int16)).cuda().view(torch.bfloat16)[:, :k], xt, s)
        want = S.gemv(np.ascontiguousarray(codes[at, :k]), x, to_plan(s.with_(rows_per_wg=1)), a_format="bf16")
    else:
        codes, scale = synthetic.quantise_fp8_rows(A)
        y = dp.gemv(torch.from_numpy(codes).cuda()[:, :k], xt, s,
                    row_scale=torch.from_numpy(scale).cuda())
        want = S.gemv(np.ascontiguousarray(codes[at, :k]), x, to_plan(s.with_(rows_per_wg=1)), a_format="fp8",
                      scale=scale[at])
    assert_same_bits(y.cpu().numpy()[at], want, (kind, m, k, s))


# (matrix type, lanes, rows): with 8 bf16 or 16 fp8 lanes per thread, the last
# row counts below and the first at or above each change of the launch
CASES = [("bf16", 512, m) for m in (1, 63, 4095, 4097, 16383, 16387)] + \
        [("bf16", 64, 130), ("bf16", 16, 70), ("bf16", 2048, 9)] + \
        [("fp8", 512, m) for m in (1, 63, 3071, 3075, 8191, 8193, 16383, 16385)] + \
        [("fp8", 64, 130), ("fp8", 16, 70), ("fp8", 4096, 9)]


@pytest.mark.parametrize("kind,L,m,steps", [(*c, steps) for c in CASES
                                             for steps in (1, 2.4, 3, 7.6, 17.01)
                                             if c[1] * c[2] * steps < 3e7])
def test_rows(kind, L, m, steps):
    k = max(1, int(L * steps))
    s = dp.Strategy(seq_len=-(-k // L), local_size=L, order=dp.STRIDED)
    check(kind, m, k, s, -(-k // 16) * 16)


@pytest.mark.parametrize("kind,L", (("bf16", 64), ("fp8", 64)))
@pytest.mark.parametrize("combine", (dp.TREE, dp.SEQ))
@pytest.mark.parametrize("max_grid", (0, 2))
def test_row_parts_and_bounded_grids(kind, L, combine, max_grid):
    s = dp.Strategy(seq_len=11, local_size=L, order=dp.STRIDED, wg_combine=combine, row_parts=2,
                    max_grid=max_grid)
    check(kind, 75, 11 * L + 13, s, 1504)
