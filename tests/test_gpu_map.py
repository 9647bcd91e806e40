"""scal at the edges of its 4-element pieces and 1,024-element work-groups, with
the launch bounded (work-groups that stride) or not, out of place and in
place.  One rounded product per element: equal bit for bit."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1710_08332_amd as dp  # noqa: E402


@pytest.mark.parametrize("n", (1, 3, 4, 5, 1023, 1024, 1025, 1027, 5000, 100003))
@pytest.mark.parametrize("max_grid", (0, 1, 3))
def test_scal_edges(n, max_grid):
    x = np.random.default_rng(n).standard_normal(n + 8, dtype=np.float32)
    s = dp.Strategy(seq_len=64, local_size=256, max_grid=max_grid)
    want = np.float32(0.3) * x[:n]
    xt = torch.from_numpy(x).cuda()
    y = torch.full((n + 8,), 7.0, device="cuda")
    dp.scal(0.3, xt[:n], s, y=y[:n])
    assert np.array_equal(y[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert bool((y[n:] == 7.0).all())              # nothing is written past the end
    dp.scal(0.3, xt[:n], s, y=xt[:n])
    got = xt.cpu().numpy()
    assert np.array_equal(got[:n].view(np.uint32), want.view(np.uint32))
    assert np.array_equal(got[n:], x[n:])
