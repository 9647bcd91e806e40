"""Which kernel a strategy leads to, where the choice is between kernels of the
same results: looked at without a GPU, on a device of 256 compute units."""

import paper_1710_08332_amd as dp
from tests.launches import launches

ACCUMS = {"plain": dp.PLAIN, "kahan": dp.KAHAN, "sum2": dp.SUM2}


def first_kernels(calls):
    """(call, its first launch) for every call."""
    made = launches(calls)
    for c, m in zip(calls, made):
        assert isinstance(m, list) and m, (c, m)
    return list(zip(calls, (m[0] for m in made)))


def test_lanes_that_do_not_fit_256_threads_keep_their_own_batches():
    # teams of 257 to 1,023 threads: 64 steps of loads would be all their registers
    calls = [(op, dict(seq_len=C, local_size=L, order=dp.STRIDED, wg_combine=dp.SEQ,
                       accum=ACCUMS[acc], final_f64=f64, passes=1), dict(n=C * L * G, dtype=dt))
             for op, acc, f64, dt in (("dot", "plain", 0, dp.F32), ("dot", "plain", 0, dp.I32),
                                      ("dot", "kahan", 0, dp.F32), ("dot", "kahan", 1, dp.F32),
                                      ("dot", "sum2", 0, dp.F32), ("asum", "plain", 0, dp.F32))
             for L in (514, 518, 770, 1022, 257, 385, 1023) for C, G in ((64, 20), (256, 60))]
    for call, l in first_kernels(calls):
        assert l["block"] > 256 and "Deep<" not in l["kernel"], (call, l)


def test_few_strided_lanes_are_one_to_a_thread():
    calls = [(op, dict(seq_len=256, local_size=L, order=dp.STRIDED, passes=1,
                       wg_combine=dp.TREE if L & (L - 1) == 0 else dp.SEQ, accum=ACCUMS[acc]),
              dict(n=256 * L * G, dtype=dt))
             for op, acc, dt in (("dot", "plain", dp.F32), ("dot", "plain", dp.I32),
                                 ("dot", "kahan", dp.F32), ("dot", "sum2", dp.F32),
                                 ("asum", "plain", dp.F32))
             for L, G in ((48, 700), (64, 1000), (66, 700), (130, 400), (256, 200), (512, 60), (1024, 40))]
    for call, l in first_kernels(calls):
        L = call[1]["local_size"]
        nv = 1 if L <= 256 else L // 256
        if "fed_reduce_kernel" not in l["kernel"]:      # (loader wavefronts: few chunks)
            assert "Deep<" in l["kernel"] and f", 1, {nv}, " in l["kernel"], (call, l)
        assert l["block"] <= 320, (call, l)


def test_every_build_for_few_lanes_can_be_launched():
    # the library holds the deep batches' kernels for strided scalar lanes in
    # teams of at most 256 threads only: order 1, 1, 2 or 4 lanes a thread, no vectors
    import re
    import subprocess
    from paper_1710_08332_amd import _lib
    names = subprocess.run(["nm", "-DC", "--defined-only", _lib.LIB_PATH], capture_output=True,
                           text=True, check=True).stdout.splitlines()
    deep = {m.group(1) for n in names
            for m in [re.search(r"reduce_kernel<dpia::Deep<dpia::\w+>, ([^>]*)>", n)] if m}
    assert deep
    for shape in deep:
        order, nv, _, _, vec, threads, staged = (v.strip() for v in shape.split(","))
        assert (order, vec, threads, staged) == ("1", "1", "256", "false") and nv in "124", shape
    rows = {m.group(1) for n in names
            for m in [re.search(r"gemv_kernel<dpia::GemvF32Acc<float, dpia::DecodeF32, 64, -1>, ([^>]*)>", n)]
            if m}
    assert rows == {f"1, 1, {combine}, 256, false" for combine in (0, 1)}


def test_short_strided_lanes_keep_four_to_a_thread():
    # the whole of a lane is in flight as it is; one lane a thread only adds
    # work-groups, and their arrivals in one pass
    G = dict(order=dp.STRIDED, wg_combine=dp.TREE)
    short = [("gemv", dict(seq_len=C, local_size=L, **G), dict(m=m, k=C * L))
             for m, L in ((64, 16), (256, 64), (1024, 64), (4096, 16)) for C in (4, 8, 16, 24)]
    short += [(op, dict(seq_len=C, local_size=L, passes=1, **G), dict(n=C * L * n))
              for op in ("dot", "asum") for C in (4, 8, 16) for L, n in ((16, 64), (64, 256), (256, 64))]
    short += [("asum", dict(seq_len=8, local_size=64, passes=2, **G), dict(n=1 << 22)),
              ("asum", dict(seq_len=32, local_size=256, passes=1, **G), dict(n=32 * 256 * 512))]
    for call, l in first_kernels(short):
        assert "Deep<" not in l["kernel"] and "float, dpia::DecodeF32, 64" not in l["kernel"], (call, l)
    long = [("gemv", dict(seq_len=C, local_size=L, **G), dict(m=m, k=C * L))
            for m, L, C in ((64, 16, 32), (256, 64, 32), (1024, 64, 64), (4096, 16, 32))]
    for call, l in first_kernels(long):
        assert "float, dpia::DecodeF32, 64" in l["kernel"], (call, l)

    # narrow teams: so many chunks to a work-group, so few work-groups
    for L, least in ((4, 64), (8, 64), (16, 128), (32, 192)):
        for lanes, deep in ((least * 256 - L, False), (least * 256, True), (60000 // L * L, True)):
            calls = [(op, dict(seq_len=C, local_size=L, passes=1, **G), dict(n=C * lanes))
                     for op in ("dot", "asum") for C in (2, 8, 24)]
            for call, l in first_kernels(calls):
                assert ("Deep<" in l["kernel"]) == deep, (call, l)
    # wide ones: work-groups enough
    for lanes, deep in ((384 * 256, True), (384 * 256 + 64, False), (1 << 18, False)):
        calls = [("asum", dict(seq_len=C, local_size=64, passes=1, **G), dict(n=C * lanes)) for C in (32, 63)]
        for call, l in first_kernels(calls):
            assert ("Deep<" in l["kernel"]) == deep, (call, l)


def test_one_pass_launches_of_short_lanes_hold_256_threads():
    # 256 chunks of 64 lanes: 64 work-groups to arrive, not 256
    calls = [(op, dict(seq_len=32, local_size=64, order=dp.STRIDED, passes=p), dict(n=32 * 64 * 256))
             for op in ("dot", "asum") for p in (1, 2)]
    calls += [(op, dict(seq_len=128, local_size=16, order=dp.CONTIGUOUS, passes=p),
               dict(n=128 * 16 * 256)) for op in ("dot", "asum") for p in (1, 2)]
    for call, l in first_kernels(calls):
        assert l["grid"] == (64 if call[1]["passes"] == 1 else 256), (call, l)


def test_contiguous_lanes_shorter_than_a_row_tile_stay_staged():
    C = dict(order=dp.CONTIGUOUS, wg_combine=dp.TREE)
    staged = [("gemv", dict(seq_len=c, local_size=L, **C), dict(m=m, k=c * L))
              for m, c, L in ((1024, 32, 16), (1024, 64, 32), (512, 64, 64), (64, 32, 64), (759, 32, 64))]
    staged += [(op, dict(seq_len=c, local_size=L, passes=p, **C), dict(n=c * L * n))
               for op in ("dot", "asum") for p in (1, 2)
               for c, L, n in ((32, 16, 256), (64, 32, 256), (64, 64, 512), (128, 64, 1000))]
    for call, l in first_kernels(staged):
        assert "rows" not in l["kernel"], (call, l)
    rows = [("gemv", dict(seq_len=c, local_size=L, **C), dict(m=m, k=k, lda=-(-k // 4) * 4))
            for m, c, L, k in ((1024, 96, 16, 1536), (256, 64, 32, 2048), (256, 32, 16, 131),
                               (759, 64, 64, 4096))]
    rows += [(op, dict(seq_len=c, local_size=L, passes=2, **C), dict(n=c * L * n))
             for op in ("dot", "asum") for c, L, n in ((96, 16, 256), (128, 32, 64), (384, 64, 1000))]
    for call, l in first_kernels(rows):
        assert "rows" in l["kernel"], (call, l)
    # (dots of few lanes from 64 elements: up to 8 lanes per compute unit in one
    # pass, 24 in two)
    for G, passes in ((128, (1, 2)), (129, (2,)), (384, (2,)), (385, ())):
        calls = [("dot", dict(seq_len=64, local_size=16, passes=q, **C), dict(n=64 * 16 * G)) for q in (1, 2)]
        for call, l in first_kernels(calls):
            assert ("rows" in l["kernel"]) == (call[1]["passes"] in passes), (G, call, l)


CODES = {dp.BF16: "GemvF32Acc<unsigned short, dpia::DecodeBF16, {e}, -1>",
         dp.FP8_E4M3: "GemvF32Acc<unsigned char, dpia::DecodeFP8, {e}, -1>"}

# (matrix type, rows, elements of a lane, lanes) where the launch changes: rows
# per team, elements per batch (0: 16)
BLOCK_LINES = [
    (dp.BF16, 8192, 7, 16, 1, 64), (dp.BF16, 8193, 7, 16, 2, 0), (dp.BF16, 8193, 8, 16, 1, 64),
    (dp.BF16, 1536, 17, 512, 1, 64), (dp.BF16, 1537, 17, 512, 2, 0), (dp.BF16, 4096, 17, 256, 1, 64),
    (dp.BF16, 4097, 17, 256, 2, 0), (dp.BF16, 15872, 17, 512, 2, 0), (dp.BF16, 15873, 17, 512, 4, 0),
    (dp.BF16, 16384, 17, 512, 4, 0), (dp.BF16, 16385, 17, 512, 2, 0), (dp.BF16, 20479, 13, 512, 2, 0),
    (dp.BF16, 20480, 13, 512, 4, 0), (dp.BF16, 20480, 12, 512, 2, 0), (dp.BF16, 40960, 17, 256, 2, 0),
    (dp.FP8_E4M3, 3072, 17, 512, 1, 64), (dp.FP8_E4M3, 3074, 17, 512, 2, 64),
    (dp.FP8_E4M3, 4096, 17, 512, 2, 64), (dp.FP8_E4M3, 4098, 17, 512, 4, 64),
    (dp.FP8_E4M3, 8192, 15, 512, 4, 64), (dp.FP8_E4M3, 8194, 19, 512, 4, 0),
    (dp.FP8_E4M3, 65552, 17, 64, 4, 64), (dp.FP8_E4M3, 32776, 17, 128, 4, 0),
    (dp.FP8_E4M3, 16388, 63, 256, 4, 0), (dp.FP8_E4M3, 16388, 64, 256, 4, 64),
    (dp.FP8_E4M3, 32768, 32, 256, 4, 0), (dp.FP8_E4M3, 32772, 32, 256, 4, 64),
    (dp.FP8_E4M3, 16386, 15, 512, 4, 0), (dp.FP8_E4M3, 16386, 16, 512, 4, 64),
    (dp.FP8_E4M3, 22528, 17, 512, 4, 64), (dp.FP8_E4M3, 22530, 17, 512, 4, 0),
    (dp.FP8_E4M3, 8194, 17, 1024, 4, 0), (dp.FP8_E4M3, 24576, 33, 512, 4, 64),
    (dp.FP8_E4M3, 24578, 33, 512, 4, 0), (dp.FP8_E4M3, 32768, 18, 512, 4, 0),
    (dp.FP8_E4M3, 24576, 18, 512, 4, 64), (dp.FP8_E4M3, 24578, 18, 512, 4, 0),
    (dp.FP8_E4M3, 65552, 15, 64, 4, 0), (dp.FP8_E4M3, 98304, 15, 64, 4, 0),
    (dp.FP8_E4M3, 98320, 15, 64, 4, 64),
    (dp.FP8_E4M3, 32770, 18, 512, 4, 64), (dp.FP8_E4M3, 36864, 18, 512, 4, 64),
    (dp.FP8_E4M3, 36866, 18, 512, 4, 0),
]


def test_row_blocks_of_codes():
    calls = [("gemv", dict(seq_len=C, local_size=L, order=dp.STRIDED), dict(dtype=dt, m=m, k=L * C))
             for dt, m, C, L, _, _ in BLOCK_LINES]
    for (call, l), (dt, m, C, L, rows, e) in zip(first_kernels(calls), BLOCK_LINES):
        nv = 8 if dt == dp.BF16 else 16
        want = f"gemv_block_kernel<dpia::{CODES[dt].format(e=e)}, {nv}, 0, {rows}>"
        assert want in l["kernel"], (call, l)


def test_strided_rows_in_halves_need_sixteen_wavefronts_per_compute_unit():
    for L in (64, 128):
        for waves, halves in ((2048, False), (3584, False), (3839, False), (3840, True), (9000, True)):
            calls = [("gemv", dict(seq_len=C, local_size=L, order=dp.STRIDED), dict(m=waves * 256 // L, k=L * C))
                     for C in (64, 100)]
            for call, l in first_kernels(calls):
                assert ("gemv_block_kernel" in l["kernel"]) == halves, (waves, call, l)


def test_fp8_rows_outside_the_blocks_have_deep_batches_where_lanes_are_long():
    # (lanes no 16 of which are whole, contiguous rows, teams of more than 256)
    for C, e in ((63, 0), (64, 64), (171, 64)):
        calls = [("gemv", dict(seq_len=C, local_size=L, order=o, wg_combine=dp.SEQ),
                  dict(dtype=dp.FP8_E4M3, m=512, k=L * C, lda=-(-L * C // 16) * 16))
                 for o, L in ((dp.STRIDED, 8), (dp.STRIDED, 24), (dp.STRIDED, 8192), (dp.STRIDED, 1),
                              (dp.CONTIGUOUS, 64), (dp.CONTIGUOUS, 300))]
        for call, l in first_kernels(calls):
            assert f"gemv_kernel<dpia::{CODES[dp.FP8_E4M3].format(e=e)}" in l["kernel"], (call, l)


def test_work_groups_of_a_bounded_grid_are_large():
    # a wavefront, or a 16-byte piece a thread, to a work-group leaves a bound
    # of a few hundred work-groups with little in flight
    def calls(g):
        return [("gemv", dict(seq_len=64, local_size=64, max_grid=g), dict(m=16384, k=4096)),
                ("gemv", dict(seq_len=256, local_size=32, max_grid=g), dict(m=8192, k=8192)),
                ("gemv", dict(seq_len=64, local_size=128, max_grid=g), dict(dtype=dp.BF16, m=8192, k=8192)),
                ("gemv", dict(seq_len=64, local_size=64, max_grid=g), dict(dtype=dp.FP8_E4M3, m=16384, k=4096)),
                ("gemv", dict(seq_len=32, local_size=512, order=dp.STRIDED, max_grid=g),
                 dict(dtype=dp.BF16, m=16384, k=16384)),
                ("gemv", dict(seq_len=64, local_size=256, order=dp.STRIDED, max_grid=g),
                 dict(dtype=dp.FP8_E4M3, m=16384, k=16384)),
                ("gemv", dict(seq_len=64, local_size=128, order=dp.STRIDED, max_grid=g), dict(m=8192, k=8192)),
                ("gemv", dict(seq_len=1024, local_size=16, max_grid=g), dict(m=256, k=16384)),
                ("dot", dict(seq_len=256, local_size=16, max_grid=g), dict(n=1 << 20)),
                ("scal", dict(seq_len=64, local_size=256, max_grid=g), dict(n=1 << 24))]
    for call, l in first_kernels(calls(60)):
        assert l["block"] == 256 and l["grid"] <= 60, (call, l)
    assert "scal_bound_kernel" in first_kernels(calls(60))[-1][1]["kernel"]
    assert all(l["block"] <= 128 for _, l in first_kernels(calls(0))[:8])
    # few strided lanes: four to a thread under a bound
    few = [("gemv", dict(seq_len=64, local_size=16, order=dp.STRIDED, max_grid=g), dict(m=4096, k=1024))
           for g in (0, 60)]
    for (call, l), lanes in zip(first_kernels(few), (1, 4)):
        assert f"-1>, 1, {lanes}, 0, 256, false>" in l["kernel"], (call, l)
    # few fp8 rows: one to a team, two under a bound
    few = [("gemv", dict(seq_len=64, local_size=64, order=dp.STRIDED, max_grid=g),
            dict(dtype=dp.FP8_E4M3, m=4096, k=4096)) for g in (0, 60)]
    for (call, l), rows in zip(first_kernels(few), (1, 2)):
        assert f", 16, 0, {rows}>" in l["kernel"], (call, l)


def test_a_fold_takes_sixteen_wavefronts_beyond_one_block_of_four():
    # a lane holds 16 values, or 8 pairs
    for acc, most in (("plain", 4096), ("kahan", 2048), ("sum2", 2048)):
        calls = [("fold", dict(seq_len=4, local_size=1, wg_combine=dp.SEQ, accum=ACCUMS[acc]),
                  dict(n=4 * G)) for G in (most, most + 1)]
        assert [l["block"] for _, l in first_kernels(calls)] == [256, 1024], acc


def test_chunks_of_long_strided_lanes_are_fed_whole_or_not():
    calls = [(op, dict(seq_len=1024, local_size=L, order=dp.STRIDED, wg_combine=dp.TREE),
              dict(n=3 * 1024 * L + r)) for op in ("dot", "asum") for L in (16, 64, 256)
             for r in (0, 1, 1024 * L - 1)]
    for call, l in first_kernels(calls):
        assert "fed_reduce_kernel" in l["kernel"], (call, l)


def test_whole_contiguous_chunks_of_64_lanes_are_fed():
    # a last chunk in part would be one wavefront's: 16 rows to a wavefront then
    for op, C, Gs in (("dot", 256, (2, 64, 128, 255)), ("dot", 512, (129, 255)), ("asum", 512, (2, 64, 255))):
        calls = [(op, dict(seq_len=C, local_size=64, passes=p, order=dp.CONTIGUOUS, wg_combine=dp.TREE),
                  dict(n=64 * C * G - r)) for G in Gs for p in (1, 2) for r in (0, 1, 64 * C - 1)]
        for call, l in first_kernels(calls):
            whole = call[2]["n"] % (64 * C) == 0
            assert ("fed_reduce_kernel" if whole else "rows_reduce_kernel") in l["kernel"], (call, l)


def test_row_blocks_hold_all_rows_of_a_sequential_combine():
    calls, need = [], []
    for dt, nv, ws in ((dp.BF16, 8, (100, 3000, 16500)), (dp.FP8_E4M3, 16, (100, 1700, 2300, 9000))):
        for w in ws:
            for team in (1, 2, 3, 4, 24, 63, 64, 128, 255, 256):
                for g in (0, 70):
                    calls.append(("gemv", dict(seq_len=2, local_size=team * nv, order=dp.STRIDED,
                                               wg_combine=dp.SEQ, max_grid=g),
                                  dict(dtype=dt, m=w * 64 // team + 1, k=2 * team * nv)))
                    need.append((team, nv))
    for (call, l), (team, nv) in zip(first_kernels(calls), need):
        rows = int(l["kernel"].split(">(")[0].rsplit(",", 1)[1])
        assert f", {nv}, 1, {rows}>" in l["kernel"] and l["block"] % team == 0, (call, l)
        # (a row's lanes and a slot for its first part)
        assert l["block"] // team * rows * (team * nv + 1) * 4 <= l["lds"] <= 160 * 1024, (call, l)
