"""Folds whose values are all held by one wavefront: from 513 values on a dot's
go lane by lane, an asum's are scanned.  One sign, the other, one value of the
other sign at either end, zeros of both signs, and the last work-group of a
launch with few and more values.  Against the additions one by one, bit for
bit."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402
from tests.test_gpu_fold import F, pairs, plain, same, values  # noqa: E402
from tests.test_gpu_thin import run  # noqa: E402


def signed(kind, n):
    v = np.abs(values("normal", n))
    if kind == "negative":
        return -v
    if kind == "first":
        v[0] = -v[0]
    elif kind == "last":
        v[-1] = -v[-1]
    elif kind == "minus zeros":
        v[::2] = F(-0.0)
    elif kind == "mixed":
        v = values("normal", n)
    return v


@pytest.mark.parametrize("kind", ("positive", "negative", "first", "last", "minus zeros", "mixed"))
@pytest.mark.parametrize("op", (dp.OP_DOT, dp.OP_ASUM))
@pytest.mark.parametrize("n", (511, 512, 513, 600, 1008, 1023, 1024, 1025))
def test_plain(kind, op, n):
    v = signed(kind, n)
    s = dp.Strategy(seq_len=4, local_size=1, wg_combine=dp.SEQ)
    got = dp.fold(op, s, torch.from_numpy(v).cuda(), 4 * n, dp.F32)
    same(got.cpu().numpy(), plain(v), (kind, op, n))


@pytest.mark.parametrize("op", ("dot", "asum"))
@pytest.mark.parametrize("G", (1, 15, 16, 17, 511, 512, 513, 1023, 1024, 1025))
def test_last_work_group(op, G):
    run(op, 3 * 16 * G, dp.Strategy(seq_len=3, local_size=16, order=dp.STRIDED, wg_combine=dp.TREE,
                                    passes=1), 7)


@pytest.mark.parametrize("kind", ("positive", "first", "mixed"))
@pytest.mark.parametrize("n", (127, 128, 129, 200, 256, 258, 511, 512))
@pytest.mark.parametrize("accum,f64", ((dp.KAHAN, 0), (dp.KAHAN, 1), (dp.SUM2, 0)))
def test_pairs(kind, n, accum, f64):
    v = signed(kind, n)
    p = np.stack([v, values("normal", n, 11) * F(2.0 ** -24) * v], axis=1)
    s = dp.Strategy(seq_len=4, local_size=1, wg_combine=dp.SEQ, accum=accum, final_f64=f64)
    got = dp.fold(dp.OP_DOT, s, torch.from_numpy(p).cuda(), 4 * n, dp.F32)
    same(got.cpu().numpy(), pairs(p[:, 0], p[:, 1], accum == dp.KAHAN, f64), (kind, n, accum, f64))
