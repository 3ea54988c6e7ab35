"""Grid sorts on either side of the size from which dense cells of up to 256 points
are ordered by waves: cells around the sizes at which the ways part."""
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


SIZES = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 258, 511, 600]


@pytest.mark.parametrize("n", [32_767, 32_768, 50_000])
@pytest.mark.parametrize("spread", ["box", "plane", "point"])
@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_cells_of_chosen_sizes_in_sorts_of_either_kind(dt, spread, n):
    rng = np.random.default_rng(n)
    g = list(vt.grid_plan(n).g)
    left, parts, i = n, [], 0
    while left > 0:
        k = min(SIZES[i % len(SIZES)], left)
        c = np.array([i % g[0], i // g[0] % g[1], i // (g[0] * g[1]) % g[2]])
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
    assert len(recs) == int(np.sum(np.diff(starts) > 16))
    for c, (off, ns) in recs.items():
        ids = sid[want[starts[c]:starts[c + 1]]]
        assert np.array_equal(sst[off + 16:off + 16 + ns + 1], np.searchsorted(ids, np.arange(ns + 1))), c
