"""Launches of the largest calls: HIP takes fewer than 2^32 work-items in a
dimension of a launch, so a call of any size has to stay below that (the
kernels stride over the rest)."""

import paper_1710_08332_amd as dp
from tests.launches import launches

HUGE_GRID = (1 << 32) - 1     # a bound on the grid that bounds nothing

GEMV = dict(seq_len=64, rows_per_wg=1)
CALLS = [
    # scal: 2^34 elements were the first too many work-items of 4 elements
    *[("scal", dict(seq_len=64, local_size=256, max_grid=g), dict(n=n))
      for n in ((1 << 34) - 1, 1 << 34, 1 << 36) for g in (0, HUGE_GRID)],
    # row-blocked codes: a work-group of 256 threads for 4 rows
    *[("gemv", dict(order=dp.STRIDED, local_size=L, max_grid=g, **GEMV), dict(dtype=dt, m=m, k=16))
      for dt, L in ((dp.BF16, 2048), (dp.FP8_E4M3, 4096), (dp.BF16, 64), (dp.FP8_E4M3, 64))
      for m in ((1 << 26) - 4, 1 << 26, 1 << 30) for g in (0, HUGE_GRID)],
    # long strided binary32 rows in halves
    *[("gemv", dict(order=dp.STRIDED, local_size=L, max_grid=g, **GEMV), dict(m=m, k=4))
      for L in (64, 128) for m in (1 << 26, 1 << 28, 1 << 30) for g in (0, HUGE_GRID)],
    # contiguous rows of many lanes, and the rows of the other kernels
    *[("gemv", dict(order=o, local_size=L, max_grid=g, **GEMV), dict(dtype=dt, m=1 << 31, k=k))
      for o, L, k in ((dp.CONTIGUOUS, 512, 4096), (dp.CONTIGUOUS, 64, 16), (dp.STRIDED, 256, 16),
                      (dp.STRIDED, 2, 128), (dp.STRIDED, 1, 64))
      for dt in (dp.F32, dp.BF16, dp.FP8_E4M3, dp.I32) for g in (0, HUGE_GRID)],
    # reductions: contiguous lanes 64 rows to a wavefront, staged, strided
    *[(op, dict(order=o, seq_len=32, local_size=L, passes=p, max_grid=g), dict(n=1 << 45))
      for op in ("dot", "asum") for o in (dp.CONTIGUOUS, dp.STRIDED) for L in (16, 64, 512, 1024)
      for p in (1, 2) for g in (0, HUGE_GRID)],
]


def test_no_launch_of_2_to_the_32_work_items():
    for (entry, strategy, args), made in zip(CALLS, launches(CALLS)):
        assert isinstance(made, list) and made, (entry, strategy, args, made)
        for l in made:
            assert 0 < l["grid"] and l["grid"] * l["block"] < 1 << 32, (entry, strategy, args, l)
