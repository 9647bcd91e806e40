"""The work this library is used for, as cases that can be timed.

Each case is one call a program makes with its operands already in device
memory and its strategy, workspace, plan and output buffers already made:
dot, asum, scal and gemv under strategies of both lane orders, the paper's
uncombined float4 form, compensated dots, bf16 and fp8 matrices, the BLAS form
of gemv, and many uneven instances in one batch.

    listed()            the cases, smallest first
    draw(rng)           another case of the same ranges
    prepare(case, seed) operands (from the seed) and what the program keeps
    run(state)          one pass; returns its outputs
    work(case)          bytes and operations the pass cannot do without
    exact(case, seed)   the outputs in 64 bits, without the library
"""

from __future__ import annotations

import math
import random

import torch

import paper_1710_08332_amd as dp

ORDERS = {"contiguous": dp.CONTIGUOUS, "strided": dp.STRIDED}
COMBINES = {"tree": dp.TREE, "seq": dp.SEQ, "none": dp.NONE}
ACCUMS = {"plain": dp.PLAIN, "kahan": dp.KAHAN, "sum2": dp.SUM2}
CODES = {"f32": dp.F32, "i32": dp.I32, "bf16": dp.BF16, "fp8": dp.FP8_E4M3}
BYTES = {"f32": 4, "i32": 4, "bf16": 2, "fp8": 1}


def listed():
    return [
        # A serving loop's small dot: a few thousand elements, a length no
        # chunk divides.  Latency, launches and the host side of a call.
        dict(name="dot_4k", op="dot", dtype="f32", n=4099, seq_len=16, local_size=64,
             order="strided", combine="tree", passes=1),
        # The small configuration: N = 2^20, split 4096 / 256, LDS tree, the
        # chunk values folded by a second pass.
        dict(name="dot_1m", op="dot", dtype="f32", n=1 << 20, seq_len=256, local_size=16,
             order="contiguous", combine="tree", passes=2),
        # A BLAS gemv as a solver's inner loop has it: y := alpha A x + beta y
        # on a matrix of no round size, rows padded to 16 bytes.
        dict(name="gemv_blas_1500x3001", op="gemv_blas", dtype="f32", m=1500, k=3001, lda=3004,
             seq_len=96, local_size=32, order="contiguous", combine="tree", rows=4, parts=1),
        # asum over a long vector of no round length, contiguous lanes of 64
        # (the first split of the strategy sweep).
        dict(name="asum_50m", op="asum", dtype="f32", n=50_000_003, seq_len=64, local_size=256,
             order="contiguous", combine="tree", passes=2),
        # The headline gemv: a step of an iterative method on 8192^2.
        dict(name="gemv_f32_8192", op="gemv", dtype="f32", m=8192, k=8192, lda=8192, seq_len=32,
             local_size=256, order="strided", combine="tree", rows=4, parts=1),
        # Quantised matrices, as inference reads its weights: fp8 with one
        # scale per row, and bf16.
        dict(name="gemv_fp8_16384", op="gemv", dtype="fp8", m=16384, k=16384, lda=16384,
             seq_len=64, local_size=256, order="strided", combine="tree", rows=1, parts=1),
        dict(name="gemv_bf16_16384", op="gemv", dtype="bf16", m=16384, k=16384, lda=16384,
             seq_len=32, local_size=512, order="strided", combine="tree", rows=1, parts=1),
        # The headline dot: N = 2^26, one pass.
        dict(name="dot_64m", op="dot", dtype="f32", n=1 << 26, seq_len=256, local_size=1024,
             order="strided", combine="tree", passes=1),
        # The paper's dot of Sec. 6.2: float4 lanes, no work-group combine,
        # 32,768 values left to the outer fold.
        dict(name="dot_64m_uncombined", op="dot", dtype="f32", n=1 << 26, seq_len=2048,
             local_size=64, order="contiguous", combine="none", passes=2, vec=4),
        # scal, the paper's fourth benchmark: a vector scaled out of place.
        dict(name="scal_64m", op="scal", dtype="f32", n=1 << 26, seq_len=64, local_size=256,
             order="strided"),
        # The precise form: Kahan lanes and a binary64 final fold over values
        # that span eight decades.
        dict(name="dot_256m_kahan", op="dot", dtype="f32", n=1 << 28, seq_len=256,
             local_size=1024, order="strided", combine="tree", passes=2, accum="kahan", f64=1),
        # Many small problems at once: 4096 dots and asums of 2^8 to 2^20
        # elements and 512 gemvs up to 4096 on a side, one plan.
        dict(name="batch_4608", op="batch", reductions=4096, gemvs=512, max_n=1 << 20,
             max_side=4096, sizes=1715),
    ]


# ------------------------------------------------------------------ drawing

def _log(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _reduction_strategy(rng, n):
    """Lanes as a caller would choose them for a length: no longer than leaves
    a few thousand lanes, and chunks enough for a few dozen work-groups."""
    c = rng.choice([v for v in (16, 64, 128, 256, 512, 1024, 8192) if v <= max(16, n // 4096)])
    l = rng.choice([v for v in (16, 64, 256, 1024) if v <= max(16, n // (32 * c))])
    return dict(seq_len=c, local_size=l, order=rng.choice(("contiguous", "strided")))


def _draw_reduction(rng, op):
    n = _log(rng, 1 << 10, 1 << 26)
    case = dict(op=op, dtype="f32", n=n, **_reduction_strategy(rng, n))
    if op == "dot" and rng.random() < 0.15:
        case["dtype"] = "i32"
    if op != "scal":
        case["combine"] = "seq" if rng.random() < 0.15 else "tree"
        case["passes"] = rng.choice((1, 2))
    if rng.random() < 0.4:                      # whole chunks only
        w = case["seq_len"] * case["local_size"]
        case["n"] = max(1, n // w) * w
    return case


def _draw_compensated(rng):
    n = _log(rng, 1 << 16, 1 << 28)
    s = _reduction_strategy(rng, min(n, 1 << 26))
    w = s["seq_len"] * s["local_size"]
    return dict(op="dot", dtype="f32", n=max(1, n // w) * w, combine="tree",
                passes=rng.choice((1, 2)), accum=rng.choice(("kahan", "sum2")),
                f64=rng.choice((0, 1)), **s)


def _draw_uncombined(rng):
    c = rng.choice((512, 1024, 2048))
    l = rng.choice((64, 128, 256))
    order = rng.choice(("contiguous", "strided"))
    w = 4 * c * l
    return dict(op="dot", dtype="f32", n=w * rng.randint(1, (1 << 26) // w), seq_len=c,
                local_size=l, order=order, combine="none", passes=rng.choice((1, 2)), vec=4)


def _draw_gemv(rng):
    dtype = rng.choice(("f32", "f32", "f32", "bf16", "bf16", "fp8", "fp8", "i32"))
    m, k = _log(rng, 64, 16384), _log(rng, 64, 16384)
    if rng.random() < 0.4:
        m, k = 1 << round(math.log2(m)), 1 << round(math.log2(k))
    parts = rng.choice((1, 1, 2))
    l = rng.choice([v for v in (16, 32, 64, 256, 512) if v <= max(16, k // (8 * parts))])
    order = rng.choice(("contiguous", "strided", "strided"))
    c = -(-k // (l * parts))
    if order == "contiguous":
        c = -(-c // 32) * 32
    rows = 4 if m % 4 == 0 and l <= 256 and rng.random() < 0.5 else 1
    case = dict(op="gemv", dtype=dtype, m=m, k=k, lda=-(-k // 16) * 16, seq_len=c, local_size=l,
                order=order, combine="seq" if rng.random() < 0.1 else "tree", rows=rows,
                parts=parts)
    if dtype != "i32" and rng.random() < 0.25:
        case["op"] = "gemv_blas"
    return case


def draw(rng):
    kind = rng.choices(("dot", "asum", "scal", "compensated", "uncombined", "gemv", "batch"),
                       (6, 3, 1, 2, 1, 6, 1))[0]
    if kind in ("dot", "asum", "scal"):
        return _draw_reduction(rng, kind)
    if kind == "compensated":
        return _draw_compensated(rng)
    if kind == "uncombined":
        return _draw_uncombined(rng)
    if kind == "gemv":
        return _draw_gemv(rng)
    return dict(op="batch", reductions=_log(rng, 16, 4096), gemvs=_log(rng, 4, 512),
                max_n=1 << rng.randint(14, 20), max_side=_log(rng, 256, 4096),
                sizes=rng.randrange(1 << 20))


# ------------------------------------------------------------------- inputs

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _uniform_pm1(g, n):
    return torch.rand(n, generator=g, device="cuda").mul_(2).sub_(1)


def _log_uniform_signed(g, n):
    sign = torch.randint(0, 2, (n,), generator=g, device="cuda", dtype=torch.int8)
    mag = torch.rand(n, generator=g, device="cuda").mul_(8).sub_(4)
    return torch.pow(10.0, mag).mul_(sign.mul_(2).sub_(1))


def _integers(g, *shape):
    return torch.randint(-(1 << 31), 1 << 31, shape, generator=g, device="cuda",
                         dtype=torch.int64).to(torch.int32)


def _vector(case, g, n):
    if case["dtype"] == "i32":
        return _integers(g, n)
    if case.get("accum", "plain") != "plain":
        return _log_uniform_signed(g, n)
    return _uniform_pm1(g, n)


def _matrix(case, g):
    """The m x k matrix in rows of lda elements, its row scales (fp8), and x."""
    m, k, lda, dtype = case["m"], case["k"], case["lda"], case["dtype"]
    if dtype == "i32":
        return _integers(g, m, lda), None, _integers(g, k)
    a = torch.randn(m, lda, generator=g, device="cuda")
    x = _uniform_pm1(g, k)
    if dtype == "bf16":
        return a.to(torch.bfloat16), None, x
    if dtype == "fp8":
        scale = a.abs().amax(dim=1).div_(448.0)
        return a.div_(scale[:, None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn), scale, x
    return a, None, x


def _batch_sizes(case):
    r = random.Random(case["sizes"])
    n = [_log(r, 256, case["max_n"]) for _ in range(case["reductions"])]
    mk = [(r.randint(64, case["max_side"]), r.randint(64, case["max_side"]))
          for _ in range(case["gemvs"])]
    return n, mk


def _pad4(v):
    return -(-v // 4) * 4


# Strided strategies by size, as a tuner picks them per size class: short
# lanes for short vectors; a gemv row over 64 or 256 lanes.
_BATCH_RED = ((1 << 12, dp.Strategy(16, 64, dp.STRIDED)), (1 << 16, dp.Strategy(16, 256, dp.STRIDED)),
              (1 << 62, dp.Strategy(64, 256, dp.STRIDED)))
_BATCH_GEMV = ((1024, dp.Strategy(16, 64, dp.STRIDED)), (1 << 62, dp.Strategy(16, 256, dp.STRIDED)))


def _batch_operands(case, seed):
    """Per instance (x, y or None) of the reductions and (A, x) of the gemvs,
    packed into three buffers."""
    n, mk = _batch_sizes(case)
    g = _generator(seed)
    xs = _uniform_pm1(g, sum(2 * _pad4(v) for v in n))
    mats = torch.randn(sum(m * _pad4(k) for m, k in mk), generator=g, device="cuda")
    vecs = _uniform_pm1(g, sum(_pad4(k) for _, k in mk))
    red, at = [], 0
    for i, v in enumerate(n):
        p = _pad4(v)
        # dots and asums alternate
        red.append((xs[at:at + v], xs[at + p:at + p + v] if i % 2 == 0 else None))
        at += 2 * p
    gemv, at, xat = [], 0, 0
    for m, k in mk:
        p = _pad4(k)
        gemv.append((mats[at:at + m * p].view(m, p)[:, :k], vecs[xat:xat + k]))
        at, xat = at + m * p, xat + p
    return red, gemv


def _strategy(case):
    return dp.Strategy(
        seq_len=case["seq_len"], local_size=case["local_size"], order=ORDERS[case["order"]],
        wg_combine=COMBINES[case.get("combine", "tree")], passes=case.get("passes", 2),
        accum=ACCUMS[case.get("accum", "plain")], final_f64=case.get("f64", 0),
        rows_per_wg=case.get("rows", 1), row_parts=case.get("parts", 1),
        vec_width=case.get("vec", 1))


def prepare(case, seed):
    op = case["op"]
    if op == "batch":
        return _prepare_batch(case, seed)
    g = _generator(seed)
    s = _strategy(case)
    if op in ("gemv", "gemv_blas"):
        a, scale, x = _matrix(case, g)
        a = a[:, :case["k"]]
        if op == "gemv":
            y = torch.empty(case["m"], device="cuda",
                            dtype=torch.int32 if case["dtype"] == "i32" else torch.float32)
            return lambda: dp.gemv(a, x, s, y=y, row_scale=scale)
        y = _uniform_pm1(g, case["m"])          # updated in place by every pass
        return lambda: dp.gemv_blas(0.75, a, x, -0.5, y, s, row_scale=scale)
    x = _vector(case, g, case["n"])
    if op == "scal":
        y = torch.empty_like(x)
        return lambda: dp.scal(0.75, x, s, y=y)
    if op == "asum":
        ws = dp.workspace(s, dp.OP_ASUM, dp.F32, 0, case["n"])
        out = torch.empty(1, device="cuda")
        return lambda: dp.asum(x, s, out=out, ws=ws)
    y = _vector(case, g, case["n"])
    ws = dp.workspace(s, dp.OP_DOT, CODES[case["dtype"]], 0, case["n"])
    out = torch.empty(1, device="cuda", dtype=torch.float64 if case.get("f64") else x.dtype)
    return lambda: dp.dot(x, y, s, out=out, ws=ws)


def _prepare_batch(case, seed):
    red, gemv = _batch_operands(case, seed)
    strategies = [s for _, s in _BATCH_RED]
    ks = sorted({k for _, x in gemv for k in (x.numel(),)})
    rows = {}
    for k in ks:
        base = next(s for top, s in _BATCH_GEMV if k <= top)
        s = base.with_(seq_len=-(-k // base.local_size))
        if s not in strategies:
            strategies.append(s)
        rows[k] = strategies.index(s)
    values = torch.empty(len(red), device="cuda")
    ys = torch.empty(sum(_pad4(a.shape[0]) for a, _ in gemv), device="cuda").zero_()
    instances = []
    for i, (x, y) in enumerate(red):
        kind = next(j for j, (top, _) in enumerate(_BATCH_RED) if x.numel() <= top)
        d = dict(op=dp.OP_DOT if y is not None else dp.OP_ASUM, strategy=kind, x=x,
                 out=values[i:i + 1])
        if y is not None:
            d["y"] = y
        instances.append(d)
    at = 0
    for a, x in gemv:
        m = a.shape[0]
        instances.append(dict(op=dp.OP_GEMV, strategy=rows[x.numel()], A=a, x=x,
                              out=ys[at:at + m]))
        at += _pad4(m)
    plan = dp.BatchPlan(instances, strategies)
    ws = plan.workspace()
    plan.upload(ws)

    def step():
        plan.run(ws)
        return values, ys
    step.keep = (red, gemv)           # the plan holds addresses: the operands stay alive
    return step


def run(state):
    return state()


# --------------------------------------------------------------------- work

def work(case):
    op = case["op"]
    if op == "batch":
        n, mk = _batch_sizes(case)
        b = sum(4 * v * (2 if i % 2 == 0 else 1) + 4 for i, v in enumerate(n))
        b += sum(4 * (m * k + k + m) for m, k in mk)
        f = sum(2 * v if i % 2 == 0 else v for i, v in enumerate(n)) + sum(2 * m * k for m, k in mk)
        return {"bytes": b, "flops": f}
    if op in ("gemv", "gemv_blas"):
        m, k = case["m"], case["k"]
        b = BYTES[case["dtype"]] * m * k + 4 * k + 4 * m
        if case["dtype"] == "fp8":
            b += 4 * m
        if op == "gemv_blas":
            b += 4 * m
        return {"bytes": b, "flops": 2 * m * k}
    n = case["n"]
    if op == "scal":
        return {"bytes": 8 * n, "flops": n}
    return {"bytes": 4 * n * (2 if op == "dot" else 1) + 4, "flops": n * (2 if op == "dot" else 1)}


# -------------------------------------------------------------------- exact

def _sum64(n, term):
    total = torch.zeros((), dtype=torch.float64, device="cuda")
    for i in range(0, n, 1 << 24):
        total += term(slice(i, min(n, i + (1 << 24)))).sum()
    return total.reshape(1)


def _dot64(x, y):
    return _sum64(x.numel(), lambda s: x[s].double() * y[s].double())


def _asum64(x):
    return _sum64(x.numel(), lambda s: x[s].double().abs())


def _gemv64(a, x):
    x = x.double()
    return torch.cat([a[i:i + 1024].double() @ x for i in range(0, a.shape[0], 1024)])


def exact(case, seed):
    op = case["op"]
    if case.get("dtype") == "i32":
        return None                   # whole numbers modulo 2^32
    if op == "batch":
        red, gemv = _batch_operands(case, seed)
        values = torch.cat([_asum64(x) if y is None else _dot64(x, y) for x, y in red])
        ys = torch.zeros(sum(_pad4(a.shape[0]) for a, _ in gemv), dtype=torch.float64,
                         device="cuda")
        at = 0
        for a, x in gemv:
            m = a.shape[0]
            ys[at:at + m] = _gemv64(a, x)
            at += _pad4(m)
        return values, ys
    g = _generator(seed)
    if op in ("gemv", "gemv_blas"):
        a, scale, x = _matrix(case, g)
        a = a[:, :case["k"]]
        v = _gemv64(a, x)
        if scale is not None:
            v = v * scale.double()
        if op == "gemv_blas":
            v = 0.75 * v - 0.5 * _uniform_pm1(g, case["m"]).double()
        return v
    x = _vector(case, g, case["n"])
    if op == "scal":
        return 0.75 * x.double()
    if op == "asum":
        return _asum64(x)
    return _dot64(x, _vector(case, g, case["n"]))
