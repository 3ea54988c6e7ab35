"""A cell handed from the list kernel to the stream kernel has its vertices solved
again there: to the same bits as in one kernel that keeps them."""
import numpy as np
import pytest
import torch

from paper_2412_04514_amd import gen

pytestmark = pytest.mark.gpu

vt = pytest.importorskip("paper_2412_04514_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("k", [8, 24, 64])
@pytest.mark.parametrize("kind", ["uniform", "cluster"])
@pytest.mark.parametrize("dt,prec", [(np.float32, "f32"), (np.float32, "f64"), (np.float64, "f64")])
def test_handed_over_vertices_keep_their_bits(dt, prec, kind, k):
    n = 6000
    # around the origin, so that a vertex keeps its low bits beside its generator's position
    P = torch.from_numpy((getattr(gen, kind)(n, seed=9, dtype=np.float64) - 0.5).astype(dt)).cuda()
    box = ((-0.5,) * 3, (0.5,) * 3)
    a = vt.tessellate(P, box, k0=k, max_gpu_retries=0, precision=prec, vertices=True, index_space="sorted")
    assert a.stats["passes"][0]["streamed"] > n // 20
    cs, perm, srt, grid = vt.grid_sort(P, box)
    lists = vt.knn(srt, grid, cs, k, dist=prec)
    b = vt.clip_cells(srt, lists, k, box=box, precision=prec, max_vert=128, stream=True, grid=grid, cell_start=cs)
    ok = (b["status"] == 0).cpu().numpy()
    rp, xyz, pl = a.vrow_ptr.cpu().numpy(), a.vxyz.cpu().numpy(), a.vplanes.cpu().numpy()
    vc, bx, bp = b["vcount"].cpu().numpy(), b["verts"].cpu().numpy(), b["vplanes"].cpu().numpy()
    checked = differ = 0
    for s in np.flatnonzero(ok):
        if rp[s + 1] - rp[s] != vc[s]:
            continue  # (beyond the fast kernel there)
        x, p = xyz[rp[s]:rp[s + 1]], np.sort(pl[rp[s]:rp[s + 1]], axis=1)
        y, q = bx[s, :vc[s]], np.sort(bp[s, :vc[s]], axis=1)
        i, j = np.lexsort(p.T), np.lexsort(q.T)
        assert np.array_equal(p[i], q[j])
        checked += len(i)
        differ += int(np.sum(np.any(x[i].view(np.int64) != y[j].view(np.int64), axis=1)))
    assert checked > 15 * n and differ == 0
