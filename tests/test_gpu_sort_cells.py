"""Grid sort with cells of chosen sizes: around the 16 points that a cell may
hold without a sub-grid, the 64 and 256 that a wave orders in registers, and
windows of 64 cells whose points end in every place of a chunk of 64."""
import numpy as np
import pytest
import torch

from test_gpu_parity import _cells_np, _sub_records

pytestmark = pytest.mark.gpu

vt = pytest.importorskip("paper_2412_04514_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


SIZES = {
    "edges": [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 258, 511, 600],
    "small": [0, 1, 2, 16, 3, 0, 0, 15, 16, 16, 16, 16, 7, 1, 64, 0],
    "one": [16, 1, 0, 1],
}


@pytest.mark.parametrize("spread", ["box", "plane", "point"])
@pytest.mark.parametrize("sizes", sorted(SIZES))
@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_cells_of_chosen_sizes(sizes, spread, dt):
    rng = np.random.default_rng(5)
    # cells along x, all sizes in turn, on a unit grid of g cells per axis
    g = 12
    n = 2 * g ** 3  # the grid that is planned for n points has about g cells per axis
    plan = SIZES[sizes]
    left, parts, i = n, [], 0
    while left > 0:
        k = min(plan[i % len(plan)] if i < g ** 3 else left, left)
        c = np.array([i % g, i // g % g, i // g ** 2 % g])
        u = rng.random((k, 3))
        if spread == "plane":
            u[:, 1] = 0.5
        elif spread == "point":
            u[:] = 0.25 + 1e-3 * rng.integers(0, 4, (k, 3))  # many of them the same
        parts.append((c + 0.1 + 0.8 * u) / g)
        left -= k
        i += 1
    P = np.concatenate(parts).astype(dt)
    P = P[rng.permutation(n)]
    cs, perm, srt, grid = vt.grid_sort(torch.from_numpy(P).cuda())
    cid = _cells_np(P, grid)
    sst = grid.sub_start.cpu().numpy()
    sid, recs = _sub_records(P, grid, cid, sst, grid.subinfo.cpu().numpy())
    want = np.lexsort((np.arange(n), sid, cid))
    starts = np.searchsorted(cid[want], np.arange(grid.ncells + 1), side="left")
    assert np.array_equal(cs.cpu().numpy(), starts)
    assert np.array_equal(perm.cpu().numpy(), want)
    assert np.array_equal(srt.cpu().numpy()[:, :3], P[want])
    ends = 0
    for c, (off, ns) in sorted(recs.items(), key=lambda e: e[1][0]):
        ids = sid[want[starts[c]:starts[c + 1]]]
        assert np.array_equal(sst[off + 16:off + 16 + ns + 1], np.searchsorted(ids, np.arange(ns + 1))), c
        assert off >= ends  # records do not overlap
        ends = off + 16 + ns + 1
    assert ends <= len(sst)
