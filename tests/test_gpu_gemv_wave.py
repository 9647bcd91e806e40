"""Staged contiguous gemv rows whose teams are launched a wavefront (or a team) to
a work-group: the lane counts and lengths at each line of that rule, row counts
that leave rows out of the last wavefront, both combines, two row parts, rows
shorter than their lanes and bounded grids.  Against the oracle, bit for bit."""

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
    if kind == "f32":
        y = dp.gemv(torch.from_numpy(A).cuda()[:, :k], xt, s)
        want = S.gemv(np.ascontiguousarray(A[at, :k]), x, to_plan(s.with_(rows_per_wg=1)))
    elif kind == "bf16":
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


@pytest.mark.parametrize("kind", ("f32", "bf16", "fp8"))
@pytest.mark.parametrize("L,C", ((16, 64), (32, 32), (32, 160), (64, 32), (64, 128), (64, 160),
                                 (128, 32), (128, 64), (256, 32)))
@pytest.mark.parametrize("combine", (dp.TREE, dp.SEQ))
@pytest.mark.parametrize("parts,short,m,max_grid", ((1, 0, 4099, 0), (1, 37, 2305, 0),
                                                    (2, 3, 2050, 7), (2, 900, 1027, 0)))
def test_wave_work_groups(kind, L, C, combine, parts, short, m, max_grid):
    s = dp.Strategy(seq_len=C, local_size=L, row_parts=parts, wg_combine=combine,
                    max_grid=max_grid)
    k = max(1, L * C * parts - short)
    check(kind, m, k, s, -(-k // 16) * 16)
