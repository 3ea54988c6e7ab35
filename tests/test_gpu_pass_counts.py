"""The statistics of passes that are taken as one, against the passes run one by
one: each pass clips the cells that the one before left, by longer lists."""
import numpy as np
import pytest
import torch

from helpers import note
from paper_2412_04514_amd import gen

pytestmark = pytest.mark.gpu

vt = pytest.importorskip("paper_2412_04514_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _left(srt, lists, cells, k, prec, large):
    """The cells that a pass by k entries leaves: those beyond the fast kernel go
    to the large one, except in the first pass."""
    def clip(c, capacity):
        r = vt.clip_cells(srt, lists[c.long(), :k].contiguous(), k, cells=c, precision=prec, capacity=capacity)
        return r["status"]

    st = clip(cells, 0)
    over = st == vt.CELL_CAPACITY
    if large and int(over.sum()):
        st = st.clone()
        st[over] = clip(cells[over].contiguous(), 1)
    return cells[(st == vt.CELL_RADIUS) | (st == vt.CELL_CAPACITY)].contiguous()


def _ridges(n, seed):
    # points on coincident spheres around some of them: cells of many faces, and
    # distances that all but tie
    rng = np.random.default_rng(seed)
    parts = [rng.random((n, 3))]
    for m in (20, 31, 40, 55, 70):
        u = rng.standard_normal((m, 3))
        c = rng.uniform(0.2, 0.8, 3)
        parts.append(np.concatenate([[c], c + 0.02 * u / np.linalg.norm(u, axis=1, keepdims=True)]))
    return np.concatenate(parts).astype(np.float32)


def _touch(seed):
    """A cell that six planes make a box, ten more do not reach, and the next one
    touches in an edge: it is unresolved from there on, in float."""
    rng = np.random.default_rng(seed)
    h = 1.0 / 64  # (the six and the last are exact in float)
    box = h * np.array([[2, 0, 0], [-2, 0, 0], [0, 2, 0], [0, -2, 0], [0, 0, 4], [0, 0, -4]])
    around = h * (np.array([[4.2, 0, 0]] * 5 + [[-4.2, 0, 0]] * 5) + rng.uniform(-0.1, 0.1, (10, 3)))
    last = h * np.array([[0, 2, 4]])
    far = rng.random((3000, 3)) - 0.5
    far = far[np.linalg.norm(far, axis=1) > 7 * h]
    return (0.5 + np.concatenate([np.zeros((1, 3)), box, around, last, far])).astype(np.float32)


SETS = {
    "touch": lambda: _touch(8),
    "uniform": lambda: gen.uniform(20_000, seed=5, dtype=np.float32),
    "cluster": lambda: gen.cluster(30_000, seed=32, dtype=np.float32),
    "filament": lambda: gen.filament(20_000, seed=6, dtype=np.float32),
    "shells": lambda: _ridges(10_000, 7),
    # one cell each pass: no pass after the first has anything to do
    "three": lambda: gen.uniform(3, seed=1, dtype=np.float32),
}


@pytest.mark.parametrize("k0,retries", [(8, 1), (8, 3), (16, 2), (24, 1), (32, 1), (12, 2)])
@pytest.mark.parametrize("name", sorted(SETS))
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_each_pass_has_its_own_counts(prec, name, k0, retries):
    P = torch.from_numpy(SETS[name]()).cuda()
    n = len(P)
    cs, perm, srt, grid = vt.grid_sort(P)
    lists = vt.knn(srt, grid, cs, 64, dist=prec)
    got = vt.tessellate(P, k0=k0, max_gpu_retries=retries, precision=prec).stats["passes"]
    cells = torch.arange(n, dtype=torch.int32, device="cuda")
    want = []
    for i in range(retries):  # (the last pass goes on by grid rings)
        if i and not len(cells):
            break
        left = _left(srt, lists, cells, k0 * 2 ** i, prec, large=i > 0)
        want.append((k0 * 2 ** i, len(cells), len(left), 0))
        cells = left
    note(f"  {name} {prec} {k0}x{retries}: {want}")
    if name == "touch" and prec == "f32" and k0 == 8 and retries == 3:
        seed = torch.nonzero(perm == 0).to(torch.int32).flatten()
        row = lists[seed.long()]
        st = [int(vt.clip_cells(srt, row[:, :k].contiguous(), k, cells=seed, precision=prec)["status"][0])
              for k in (8, 16, 32)]
        assert st == [vt.CELL_RADIUS, vt.CELL_RADIUS, vt.CELL_UNRESOLVED]
    assert [(p["k"], p["cells"], p["failed"], p["streamed"]) for p in got[:len(want)]] == want
    if len(cells):
        assert len(got) == retries + 1 and (got[-1]["k"], got[-1]["cells"]) == (k0 * 2 ** retries, len(cells))
    else:
        assert len(got) == len(want)
