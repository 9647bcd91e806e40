"""Binary32 gemv rows where the launch changes: contiguous lanes 16, 32 or 64 to
a wavefront (from 16 to 512 lanes a row, rows that share a work-group, rows
shorter than their lanes), strided rows of few lanes one to a thread.  Against
the oracle, bit for bit."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
import synthetic  # noqa: E402
from oracle import strategies as S  # noqa: E402
from tests.gpu_util import assert_same_bits, to_plan  # noqa: E402


def check(m, k, s, lda, blas=False):
    g = synthetic.rng(m * 7 + k)
    A, x, y = synthetic.normal(g, (m, lda)), synthetic.uniform_pm1(g, k), synthetic.uniform_pm1(g, m)
    at = np.arange(m) if m <= 400 else np.unique(np.r_[np.arange(64), np.arange(m - 64, m),
                                                       g.integers(0, m, 150)])
    At, xt = torch.from_numpy(A).cuda()[:, :k], torch.from_numpy(x).cuda()
    rows, plan = np.ascontiguousarray(A[at, :k]), to_plan(s.with_(rows_per_wg=1))
    if blas:
        got = dp.gemv_blas(0.75, At, xt, -0.5, torch.from_numpy(y).cuda(), s)
        want = S.gemv_blas(0.75, rows, x, -0.5, y[at], plan)
    else:
        got, want = dp.gemv(At, xt, s), S.gemv(rows, x, plan)
    assert_same_bits(got.cpu().numpy()[at], want, (m, k, s))


@pytest.mark.parametrize("L", (16, 32, 64, 320, 512, 1024))
@pytest.mark.parametrize("C", (32, 96, 160))
@pytest.mark.parametrize("short", (0, 5, 40))          # elements missing, or most lanes
@pytest.mark.parametrize("parts", (1, 2))
def test_contiguous_rows(L, C, short, parts):
    combine = dp.SEQ if L & (L - 1) or C == 96 else dp.TREE
    s = dp.Strategy(seq_len=C, local_size=L, row_parts=parts, wg_combine=combine)
    k = L * C * parts - short if short < 40 else max(1, L * C * parts // 40)
    check(37, k, s, -(-k // 4) * 4, blas=short == 5)


@pytest.mark.parametrize("order", (dp.CONTIGUOUS, dp.STRIDED))
@pytest.mark.parametrize("L,m", ((16, 2048), (64, 512), (32, 2048), (64, 1024), (16, 4096), (256, 256)))
@pytest.mark.parametrize("off", (0, 1))
def test_lane_counts(order, L, m, off):
    s = dp.Strategy(seq_len=32, local_size=L, order=order)
    check(m + off, 32 * L - 3, s, 32 * L)


@pytest.mark.parametrize("L", (16, 48, 64, 256))
@pytest.mark.parametrize("C", (1, 63, 64, 65, 127, 161))
@pytest.mark.parametrize("parts", (1, 2))
def test_thin_strided_rows(L, C, parts):
    s = dp.Strategy(seq_len=C, local_size=L, order=dp.STRIDED, row_parts=parts,
                    wg_combine=dp.TREE if L & (L - 1) == 0 else dp.SEQ,
                    max_grid=3 if C == 65 else 0)
    k = L * C * parts - L // 3
    check(29, k, s, -(-k // 4) * 4, blas=C == 63)


# 8 wavefronts per compute unit: the batch in two halves from there on
@pytest.mark.parametrize("L,m", ((64, 8191), (64, 8192), (128, 4095), (128, 4099)))
@pytest.mark.parametrize("steps", (64, 66.5, 71))
@pytest.mark.parametrize("combine", (dp.TREE, dp.SEQ))
def test_half_batches(L, m, steps, combine):
    k = int(L * steps)
    s = dp.Strategy(seq_len=-(-k // L), local_size=L, order=dp.STRIDED, wg_combine=combine)
    check(m, k, s, -(-k // 4) * 4, blas=steps == 71)
