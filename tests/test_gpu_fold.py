"""The outer reduceSeq over the chunk values, on its own: every length around
the edges of a lane, a wavefront and a block of the fold, over values whose
running sum stays in its binade, leaves it often, meets ties, cancels to zero,
underflows, overflows or is not a number.  Expected: the additions one by one
(the stated steps of the compensated forms), each rounded; equal bit for bit,
so there is no tolerance."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402

F = np.float32


def values(kind, n, seed=7):
    g = np.random.default_rng(seed + n)
    if kind == "normal":
        return g.standard_normal(n, dtype=F)
    if kind == "positive":
        return g.random(n, dtype=F)
    if kind == "wide":                        # many binades, both signs
        return (10.0 ** g.uniform(-4, 4, n) * g.choice((-1.0, 1.0), n)).astype(F)
    if kind == "alternating":                 # a change of binade at every step
        return np.where(np.arange(n) % 2 == 0, F(1), F(-1)) + g.standard_normal(n, dtype=F) * F(1e-3)
    if kind == "ties":                        # half a unit of the running sum
        v = g.integers(-3, 4, n).astype(F) * F(0.5)
        v[0] = F(2 ** 23 + 2 ** 22)
        return v
    if kind == "edge":                        # about a power of two, from both sides
        v = g.choice((-1.0, -0.5, -0.25, 0.25, 0.5, 1.0), n).astype(F)
        v[0] = F(2 ** 23)
        return v
    if kind == "zeros":
        v = np.zeros(n, F)
        v[1::3] = F(-0.0)
        return v
    if kind == "tiny":                        # subnormal sums
        return (g.integers(-4, 5, n) * 2.0 ** -149).astype(F)
    if kind == "overflow":
        v = g.standard_normal(n, dtype=F)
        v[n // 2:] = F(3e38)
        return v
    v = g.standard_normal(n, dtype=F)
    v[n // 3] = F(np.inf)
    v[n // 2] = F(-np.inf)
    v[2 * n // 3] = F(np.nan)
    return v


KINDS = ("normal", "positive", "wide", "alternating", "ties", "edge", "zeros", "tiny", "overflow",
         "nan")


def plain(v):
    acc = F(0)
    with np.errstate(all="ignore"):
        for e in v:
            acc = F(e + acc)
    return acc


def pairs(s, c, kahan, f64):
    """The fold of compensated pairs: s - c (Kahan) or s + c (Sum2)."""
    with np.errstate(all="ignore"):
        if f64:
            acc = np.float64(0)
            for x, y in zip(s.astype(np.float64), c.astype(np.float64)):
                acc = (x - y if kahan else x + y) + acc
            return acc
        ls, lc = F(0), F(0)
        for rs, rc in zip(s, c):
            t = F(ls + rs)
            bp = F(t - ls)
            e = F(F(ls - F(t - bp)) + F(rs - bp))
            lc = F(F(lc + rc) - e) if kahan else F(F(lc + rc) + e)
            ls = t
        return F(ls - lc) if kahan else F(ls + lc)


def same(got, want, note):
    got, want = np.asarray(got).reshape(-1)[0], np.asarray(want).reshape(-1)[0]
    assert got.dtype == want.dtype, note
    assert (np.isnan(got) and np.isnan(want)) or got.tobytes() == want.tobytes(), (note, got, want)


# lanes of 16 values, 64 lanes a wavefront, 4 or (beyond 4096) 16 wavefronts
SIZES = (1, 15, 17, 511, 512, 513, 1023, 1025, 2049, 4095, 4096, 4097, 16385, 33001)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", SIZES)
def test_plain_fold(kind, n):
    v = values(kind, n)
    s = dp.Strategy(seq_len=4, local_size=1, wg_combine=dp.SEQ)
    got = dp.fold(dp.OP_DOT, s, torch.from_numpy(v).cuda(), 4 * n, dp.F32)
    same(got.cpu().numpy(), plain(v), (kind, n))


def test_chunk_values_at_any_element():
    # dpia_fold takes chunk values at any address of their type
    v = values("normal", 2501)
    s = dp.Strategy(seq_len=4, local_size=1, wg_combine=dp.SEQ)
    t = torch.from_numpy(v).cuda()
    for at in (1, 2, 3, 5):
        got = dp.fold(dp.OP_DOT, s, t[at:], 4 * (2501 - at), dp.F32)
        same(got.cpu().numpy(), plain(v[at:]), at)


@pytest.mark.parametrize("kind", ("normal", "wide", "alternating", "edge", "zeros", "nan"))
@pytest.mark.parametrize("n", (1, 7, 9, 255, 257, 513, 2047, 2049, 9001))
@pytest.mark.parametrize("accum", (dp.KAHAN, dp.SUM2))
@pytest.mark.parametrize("f64", (0, 1))
def test_compensated_fold(kind, n, accum, f64):
    v = values(kind, n)
    c = np.nan_to_num(values("normal", n, 11) * F(2.0 ** -24) * np.abs(v), posinf=0, neginf=0)
    p = np.stack([v, c.astype(F)], axis=1)
    s = dp.Strategy(seq_len=4, local_size=1, wg_combine=dp.SEQ, accum=accum, final_f64=f64)
    got = dp.fold(dp.OP_DOT, s, torch.from_numpy(p).cuda(), 4 * n, dp.F32)
    same(got.cpu().numpy(), pairs(p[:, 0], p[:, 1], accum == dp.KAHAN, f64), (kind, n, accum, f64))


@pytest.mark.parametrize("n", (1, 63, 65, 255, 257, 1025, 20001))
def test_integer_fold(n):
    v = np.random.default_rng(n).integers(-(1 << 31), 1 << 31, n).astype(np.int32)
    s = dp.Strategy(seq_len=4, local_size=1, wg_combine=dp.SEQ)
    got = dp.fold(dp.OP_DOT, s, torch.from_numpy(v).cuda(), 4 * n, dp.I32)
    want = np.uint32(int(v.astype(np.int64).sum()) & 0xFFFFFFFF)
    assert got.cpu().numpy().view(np.uint32)[0] == want


# one pass: the fold runs in the reduction's own work-group, of 64, 200, 256
# and 1024 threads
@pytest.mark.parametrize("C,L,order", ((4, 16, dp.STRIDED), (4, 64, dp.CONTIGUOUS),
                                       (8, 100, dp.CONTIGUOUS), (4, 1024, dp.CONTIGUOUS)))
@pytest.mark.parametrize("G", (3, 513, 1500, 4500))
@pytest.mark.parametrize("accum", (dp.PLAIN, dp.KAHAN))
def test_one_pass_fold(C, L, order, G, accum):
    n = C * L * G
    g = np.random.default_rng(n)
    x, y = (g.random(n, dtype=F) * F(2) - F(1) for _ in range(2))
    s = dp.Strategy(seq_len=C, local_size=L, order=order, passes=1, accum=accum,
                    wg_combine=dp.TREE if L & (L - 1) == 0 else dp.SEQ)
    xt, yt = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    c = dp.chunks(dp.OP_DOT, s, xt, yt).cpu().numpy().view(F)
    want = plain(c[:G]) if accum == dp.PLAIN else pairs(c[0:2 * G:2], c[1:2 * G:2], True, 0)
    ws = dp.workspace(s, dp.OP_DOT, dp.F32, 0, n)
    for _ in range(2):                        # the counters are left at zero
        same(dp.dot(xt, yt, s, ws=ws).cpu().numpy(), want, (C, L, order, G, accum))
