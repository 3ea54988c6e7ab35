"""k-NN lists of points so far apart that d^2 overflows: every other point is
listed all the same, in the order of (infinite d^2, sorted index)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

vt = pytest.importorskip("paper_2412_04514_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("k", [8, 12, 16, 24, 32, 48, 64, 128])
@pytest.mark.parametrize("dt,dist,scale", [(np.float64, "f64", 1e160), (np.float32, "f32", 1e25)])
def test_points_beyond_the_range_of_d2_are_listed(dt, dist, scale, k):
    n = 45
    P = (np.random.default_rng(6).uniform(-1, 1, (n, 3)) * scale).astype(dt)
    box = ((-scale,) * 3, (scale,) * 3)
    grid = vt.grid_plan(1, box)  # one cell
    cs, perm, srt, grid = vt.grid_sort(torch.from_numpy(P).cuda(), box, grid=grid)
    got = vt.knn(srt, grid, cs, k, dist=dist).cpu().numpy()
    S = srt[:, :3].cpu().numpy()
    with np.errstate(over="ignore"):
        for i in range(n):
            x = S - S[i]
            d2 = (x[:, 0] * x[:, 0] + x[:, 1] * x[:, 1]) + x[:, 2] * x[:, 2]
            order = [j for j in np.lexsort((np.arange(n), d2)) if j != i]
            assert np.isinf(d2).sum() >= n - 3
            want = (order + [-1] * k)[:k]
            assert got[i].tolist() == want
