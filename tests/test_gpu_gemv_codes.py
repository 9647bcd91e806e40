"""bf16 and fp8 gemv: the row-blocked kernels on both sides of every line of
their dispatch (tests/test_launch_rules.py holds which kernel that is), with
remainders of every size of the deep batches; and the rows that are not
blocked: lanes of which no 8 or 16 are whole, one or two lanes, teams of more
than 256 threads, contiguous lanes of every vector width, whole and not.  Rows
repeat a few base rows, so that every row is compared with the oracle."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
import synthetic  # noqa: E402
from oracle import strategies as S  # noqa: E402
from tests.gpu_util import assert_same_bits, to_plan  # noqa: E402
from tests.test_launch_rules import BLOCK_LINES  # noqa: E402

BASE = 37


def check(dt, m, k, s):
    g = synthetic.rng(m + k)
    lda = -(-k // 16) * 16
    A, x = synthetic.normal(g, (BASE, lda)), synthetic.uniform_pm1(g, k)
    xt = torch.from_numpy(x).cuda()
    at = torch.arange(m, device="cuda") % BASE
    if dt == dp.BF16:
        codes = synthetic.quantise_bf16(A)
        t = torch.from_numpy(codes.view(np.int16)).cuda()[at].view(torch.bfloat16)
        y = dp.gemv(t[:, :k], xt, s)
        want = S.gemv(np.ascontiguousarray(codes[:, :k]), x, to_plan(s), a_format="bf16")
    else:
        codes, scale = synthetic.quantise_fp8_rows(A)
        t = torch.from_numpy(codes).cuda()[at]
        y = dp.gemv(t[:, :k], xt, s, row_scale=torch.from_numpy(scale).cuda()[at])
        want = S.gemv(np.ascontiguousarray(codes[:, :k]), x, to_plan(s), a_format="fp8", scale=scale)
    assert_same_bits(y.cpu().numpy(), want[np.arange(m) % BASE], (dt, m, k, s))


@pytest.mark.parametrize("dt,m,C,L", [c[:4] for c in BLOCK_LINES])
@pytest.mark.parametrize("steps,short", ((0, 0), (0, 5), (1, 40)))
def test_block_lines(dt, m, C, L, steps, short):
    check(dt, m, L * (C - steps) - short, dp.Strategy(seq_len=C, local_size=L, order=dp.STRIDED))


@pytest.mark.parametrize("C", (16, 17, 18, 19, 20, 23))
@pytest.mark.parametrize("m", (4096, 8192))
def test_remainders_of_the_deep_batch(m, C):
    check(dp.FP8_E4M3, m, 512 * C, dp.Strategy(seq_len=C, local_size=512, order=dp.STRIDED))


@pytest.mark.parametrize("dt", (dp.BF16, dp.FP8_E4M3))
@pytest.mark.parametrize("L,C", ((8, 64), (8, 171), (24, 67), (1, 130), (2, 100), (4, 90), (12, 65),
                                 (100, 64), (40, 20)))
@pytest.mark.parametrize("short", (0, 3))
def test_strided_rows_outside_the_blocks(dt, L, C, short):
    s = dp.Strategy(seq_len=C, local_size=L, order=dp.STRIDED,
                    wg_combine=dp.TREE if L & (L - 1) == 0 else dp.SEQ)
    check(dt, 75, L * C - short, s)


@pytest.mark.parametrize("dt", (dp.BF16, dp.FP8_E4M3))
@pytest.mark.parametrize("L,C", ((64, 80), (64, 72), (128, 100), (128, 66), (64, 65), (300, 64),
                                 (512, 64), (1024, 96), (512, 32), (300, 48), (16, 500)))
@pytest.mark.parametrize("short", (0, 1, 7))
def test_contiguous_rows(dt, L, C, short):
    s = dp.Strategy(seq_len=C, local_size=L, wg_combine=dp.TREE if L & (L - 1) == 0 else dp.SEQ)
    check(dt, 41, L * C - short, s)


@pytest.mark.parametrize("dt,w", [(dp.BF16, w) for w in (100, 3000, 16500)] +
                         [(dp.FP8_E4M3, w) for w in (100, 1700, 2300, 9000)])
@pytest.mark.parametrize("team", (1, 2, 3, 4, 24, 64, 256))
@pytest.mark.parametrize("parts", (1, 2))
def test_rows_combined_one_after_the_other(dt, w, team, parts):
    # a thread to each of a team's 1, 2 or 4 rows, more rows than threads among them
    L = team * (8 if dt == dp.BF16 else 16)
    s = dp.Strategy(seq_len=2, local_size=L, order=dp.STRIDED, wg_combine=dp.SEQ, row_parts=parts)
    check(dt, w * 64 // team + 1, 2 * L * parts - L - 3, s)
