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
