"""Cells far thinner than long and far smaller than the box, in double: a point
beyond the list whose bisector takes a hair off the cell's tip is a neighbour."""
from fractions import Fraction

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

vt = pytest.importorskip("paper_2412_04514_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _dot(a, b):
    return sum(x * y for x, y in zip(a, b))


def _vertex(planes):
    """Where three bisectors with the origin's point meet, exactly."""
    n = [[Fraction(float(x)) for x in p] for p in planes]
    c = [_dot(p, p) / 2 for p in n]

    def cross(a, b):
        return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]

    m = [cross(n[1], n[2]), cross(n[2], n[0]), cross(n[0], n[1])]
    det = _dot(n[0], m[0])
    return [sum(c[i] * m[i][a] for i in range(3)) / det for a in range(3)]


def _spindle(rng, R, d, dl):
    """A point in the origin, six around it at dl whose bisectors make a spindle
    with its tips at distance R, two that do not reach it, and for each tip one
    at d whose bisector cuts it by 1e-10 d R."""
    t, a, b = np.linalg.qr(rng.standard_normal((3, 3)))[0].T
    lean = dl / (2 * R)
    side = [np.sqrt(1 - lean ** 2) * (np.cos(w) * a + np.sin(w) * b) + lean * (-1) ** i * t
            for i, w in enumerate(np.arange(6) * np.pi / 3)]
    pts = [np.zeros(3)] + [dl * s for s in side] + [3 * dl * (a + b), 3 * dl * (a - b)]
    for i in (0, 1):
        v = _vertex([pts[1 + i], pts[3 + i], pts[5 + i]])
        vf = np.array([float(x) for x in v])
        w = rng.uniform(0, 2 * np.pi)
        e = d * (np.cos(w) * a + np.sin(w) * b)
        along = vf / np.linalg.norm(vf)
        for _ in range(3):  # the part of e along the tip that makes e.v = |e|^2 / 2 + 1e-10 d R
            e = e + (0.5 * (e @ e) + 1e-10 * d * R - e @ vf) / np.linalg.norm(vf) * along
        f = [Fraction(float(x)) for x in e]
        over = _dot(f, v) - _dot(f, f) / 2
        assert 0 < over < Fraction(d * R) / 10 ** 6  # it cuts, and barely
        pts.append(e)
    return np.array(pts)


@pytest.mark.parametrize("R,d", [(1e-2, 1e-5), (1e-8, 1e-11), (1e-10, 1e-13), (1e-10, 1e-12)])
def test_points_that_just_cut_a_tip(R, d):
    rng = np.random.default_rng(17)
    missing = 0
    for _ in range(100):
        P = torch.from_numpy(_spindle(rng, R, d, d / 10)).cuda()
        box = ((-1.0,) * 3, (1.0,) * 3)
        cs, perm, srt, grid = vt.grid_sort(P, box)
        cell = torch.nonzero(perm == 0).to(torch.int32).flatten()
        lists = vt.knn(srt, grid, cs, 8, queries=cell)
        r = vt.clip_cells(srt, lists, 8, box=box, cells=cell, stream=True, grid=grid, cell_start=cs)
        assert int(r["status"][0]) == 0
        nbr = perm[r["nbr"][0, :int(r["nbr_count"][0])].long()].tolist()
        assert set(range(1, 7)) <= set(nbr)
        missing += 2 - len({9, 10} & set(nbr))
    assert missing == 0
