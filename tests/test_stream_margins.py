"""The margin behind the stream phase's vertex pruning, checked in the
arithmetic the float clip uses.  A float vertex v with per-axis error bound e
stands for a true vertex c with |c_a - v_a| <= e; the ball through the seed
centred at c has radius |c| and reaches |q| <= 2 |c| from the seed.  The
kernel widens the radius to rad = |v| (1 + 1e-5) + 4 e (in float) and leaves
the vertex out when rad < rlim = float(sqrt(d_k^2 (1 - 1e-6)) / 2 (1 - 1e-6)).
Such a ball must hold list members only: 2 |c| < sqrt(d_k^2 (1 - 1e-6)), the
radius of the ball whose points are list members after the rounding of d^2."""
from pathlib import Path

import numpy as np
import pytest

f32 = np.float32


def rad_f32(v, e):
    x, y, z = (f32(t) for t in v)
    n = np.sqrt(f32(x * x + y * y) + f32(z * z), dtype=f32)
    return f32(f32(n * f32(1.0 + 1e-5)) + f32(f32(4.0) * f32(e)))


def rlim_f32(dk2):
    dk2in = float(dk2) * (1.0 - 1e-6)
    return f32(0.5 * np.sqrt(dk2in) * (1.0 - 1e-6))


def worst_c_norm(v, e):
    # the largest |c| over the box |c_a - v_a| <= e: each axis pushed away
    # from the seed
    c = np.abs(np.asarray(v, dtype=np.longdouble)) + np.longdouble(float(e))
    return np.sqrt(np.sum(c * c))


def test_pruned_balls_stay_inside_the_list_ball():
    rng = np.random.default_rng(7)
    checked = 0
    for _ in range(20000):
        v = (rng.standard_normal(3) * 10.0 ** rng.uniform(-4, 0)).astype(f32)
        e = f32(abs(v).max() * 10.0 ** rng.uniform(-8, -4.8))  # up to 16 eps |v|
        rad = rad_f32(v, e)
        # list distances from one to three radii, and just above the pruning
        # threshold, where the margin is thinnest: 2 rad (1 + s)
        ts = list(rng.uniform(1.0, 3.0, 3)) + [2.0 * (1.0 + s) for s in (1e-9, 1e-7, 1e-6, 3e-6, 1e-5)]
        for t in ts:
            dk2 = f32((float(rad) * t) ** 2)
            if not rad < rlim_f32(dk2):
                continue
            checked += 1
            assert 2 * worst_c_norm(v, e) < np.sqrt(np.longdouble(float(dk2)) * np.longdouble(1 - 1e-6))
    assert checked > 10000


def test_vertices_reaching_the_list_ball_are_kept():
    # a vertex whose true ball reaches past the list's ball is never left out
    rng = np.random.default_rng(8)
    for _ in range(20000):
        v = (rng.standard_normal(3) * 10.0 ** rng.uniform(-4, 0)).astype(f32)
        e = f32(abs(v).max() * 10.0 ** rng.uniform(-8, -4.8))
        two_c = 2 * float(np.sqrt(np.sum(np.asarray(v, np.float64) ** 2)))
        dk2 = f32((two_c * (1.0 - 1e-7)) ** 2)  # the ball of c = v reaches past it
        assert not rad_f32(v, e) < rlim_f32(dk2)


def d2_f32(q, p):
    # the clip's float d^2: each coordinate difference rounded to float, each
    # square rounded, (x^2 + y^2) + z^2 with no fused multiply-add
    dx, dy, dz = (f32(f32(a) - f32(b)) for a, b in zip(q, p))
    return f32(f32(f32(dx * dx) + f32(dy * dy)) + f32(dz * dz))


def test_float_d2_within_the_list_ball_margin():
    # a box skipped as inside the list's ball, d^2 < d_k^2 (1 - 1e-6) in exact
    # arithmetic, holds only points whose float d^2 is below the list's float
    # d_k^2: the float d^2 is within 1e-6 relative of the exact one
    rng = np.random.default_rng(9)
    p = rng.uniform(0, 1, (50000, 3)).astype(f32)
    q = (p.astype(np.float64) + rng.standard_normal((50000, 3)) * 10.0 ** rng.uniform(-5, -1, (50000, 1)))
    q = np.clip(q, 0, 1).astype(f32)
    exact = np.sum((q.astype(np.float64) - p.astype(np.float64)) ** 2, axis=1)
    got = np.array([d2_f32(a, b) for a, b in zip(q, p)], dtype=np.float64)
    keep = exact > 0
    rel = np.abs(got[keep] - exact[keep]) / exact[keep]
    assert rel.max() < 1e-6 / 2


# The float clip's windows.  A plane with normal n and offset c = |n|^2 / 2 is
# tested against a float vertex v of error bound e by s = n.v - c; where
# |s| <= eps (|n_x v_x| + |n_y v_y| + |n_z v_z| + c) + |n|_1 e the test is made
# again in double.  Three bounds on that window save tests: a plane is left out
# when max_v n.v < c - w (the list's batches; the stream's candidates), and the
# vertices are not looked at again when min_v |s| - |n|_1 e > w0.  None may leave
# out a plane that the test itself would have cut by or looked at again.
def fma32(x, y, z):  # (the product is exact in double; one more rounding of 2^-53)
    return (x.astype(np.float64) * y + z).astype(f32)


def hw_sqrt(x):  # the hardware's square root takes no denormals
    return np.where(x < np.finfo(f32).tiny, f32(0), np.sqrt(x, dtype=f32))


def dots(n, v):
    """n.v with every way of fusing that a compiler may choose."""
    (a, b, c), (x, y, z) = n.T, v.T
    yield (a * x + b * y) + c * z
    yield fma32(c, z, fma32(b, y, a * x))
    yield fma32(c, z, fma32(a, x, b * y))
    yield fma32(a, x, b * y) + c * z
    yield fma32(a, x, fma32(b, y, c * z))


def clip_constants(eps):
    verrel = np.maximum(f32(16.0) * f32(eps), np.finfo(f32).eps)
    return verrel, f32(f32(eps) + f32(1.7321) * verrel)


def radius_up(r2, eps):
    verrel, _ = clip_constants(eps)
    kap = f32((f32(3.5) + verrel) * verrel + f32(2.0) * f32(eps) + f32(4e-6))
    return r2 * (f32(1.0) + kap), kap


def list_window(d2, c, r2up, eps):
    _, wv = clip_constants(eps)
    return ((f32(eps) + f32(5e-7)) * c + (wv + f32(5e-7)) * (hw_sqrt(d2) * hw_sqrt(r2up))) * f32(1.0 + 1e-4)


def list_window0(d2, c, r2up, eps):
    return f32(eps) * (c + hw_sqrt(d2) * hw_sqrt(r2up)) * f32(1.0 + 1e-4)


def stream_window(c, r2up, eps):
    _, wv = clip_constants(eps)
    return (wv + f32(2e-6)) * (c + hw_sqrt(f32(2.0) * c) * hw_sqrt(r2up))


def hard_tests(rng, count, eps, scale, ratio):
    """Vertices at radius `scale`, planes at `ratio` of it and vertex errors at
    their bound, with s on the lower edge of the window; half of them in the
    directions where the window is largest for |n| |v|."""
    v = rng.standard_normal((count, 3))
    n = rng.standard_normal((count, 3))
    half = count // 2
    v[:half] = np.eye(3)[rng.integers(0, 3, half)] + 0.02 * rng.standard_normal((half, 3))
    n[:half] = rng.choice([-1.0, 1.0], (half, 3)) + 0.02 * rng.standard_normal((half, 3))
    v *= scale / np.linalg.norm(v, axis=1, keepdims=True)
    n *= scale * ratio / np.linalg.norm(n, axis=1, keepdims=True)
    verrel, _ = clip_constants(eps)
    e = np.abs(v).max(axis=1) * float(verrel)
    # n turned about v, so that n.v comes to the window's edge
    c = 0.5 * (n * n).sum(axis=1)
    win = eps * (np.abs(n * v).sum(axis=1) + c) + np.abs(n).sum(axis=1) * e
    u = v / scale
    along = (c - win * (1.0 - 10.0 ** rng.uniform(-9, -6, count))) / scale
    across = n - (n * u).sum(axis=1, keepdims=True) * u
    left = (scale * ratio) ** 2 - along ** 2
    ok = left > 0
    across *= (np.sqrt(np.maximum(left, 0)) / np.linalg.norm(across, axis=1))[:, None]
    n = along[:, None] * u + across
    v, n = v[ok].astype(f32), n[ok].astype(f32)
    e = (np.abs(v).max(axis=1) * verrel).astype(f32)
    return v, n, e


# (a float cell's vertices are solved from products of four lengths, which hold
# down to 1e-9 of the unit and up to 1e9)
SCALES = [(1e-9, 0.5), (1e-9, 2.0), (4e-10, 1.0), (4e-10, 2.0), (1e-6, 1e-2), (1e-4, 1e-4), (1.0, 1e-4), (1.0, 1.0), (1.0, 2.0),
          (1e9, 1.0), (3e9, 2.0)]


@pytest.mark.parametrize("eps", [1e-9, 1e-7, 1e-6, 1e-4])
@pytest.mark.parametrize("scale,ratio", SCALES)
def test_windows_hold_every_test_that_is_made_again(eps, scale, ratio):
    rng = np.random.default_rng(11)
    v, n, e = hard_tests(rng, 200_000, eps, scale, ratio)
    d2 = (n[:, 0] * n[:, 0] + n[:, 1] * n[:, 1]) + n[:, 2] * n[:, 2]
    c = f32(0.5) * d2
    r2up, _ = radius_up((v[:, 0] * v[:, 0] + v[:, 1] * v[:, 1]) + v[:, 2] * v[:, 2], eps)
    nrm1 = np.abs(n).sum(axis=1, dtype=f32)
    size = np.abs(n * v).sum(axis=1, dtype=f32) + c
    hard = 0
    for tested in dots(n, v):
        s = tested - c
        again = ~(s < -(f32(eps) * size + nrm1 * e))  # cut by, or looked at again
        near = np.abs(s) - nrm1 * f32(1.0 + 1e-6) * e <= list_window0(d2, c, r2up, eps)
        assert np.all(near[again & (s <= 0)])
        for far in dots(n, v):
            far = np.maximum(far, -c)
            assert not np.any(again & (far < c - list_window(d2, c, r2up, eps)))
            assert not np.any(again & (far < c - stream_window(c, r2up, eps)))
        hard += int(np.sum(again & (s < 0)))
    assert hard > 1000  # the edge was met
    assert np.all(np.isfinite(list_window(d2, c, r2up, eps)))  # and the bounds save something


@pytest.mark.parametrize("eps", [1e-9, 1e-6, 1e-4, 1e-2])
def test_radius_bounds_lie_within_kap(eps):
    rng = np.random.default_rng(12)
    v = rng.standard_normal((200_000, 3))
    v[::2] = rng.choice([-1.0, 1.0], (100_000, 3)) * np.array([1.0, 0.366, 0.366]) * rng.uniform(0.9, 1.1, (100_000, 3))
    v = (v * 10.0 ** rng.uniform(-8, 8, (len(v), 1))).astype(f32)
    verrel, _ = clip_constants(eps)
    e = (np.abs(v).max(axis=1) * verrel).astype(np.float64)
    w = v.astype(np.float64)
    r2 = (v[:, 0] * v[:, 0] + v[:, 1] * v[:, 1]) + v[:, 2] * v[:, 2]
    up, kap = radius_up(r2, eps)
    n1, n2 = np.abs(w).sum(axis=1), (w * w).sum(axis=1)
    margin = 1.0 - 8 * np.finfo(f32).eps  # of float lists
    # a distance above 4 up certifies the largest radius, one below 4 r2 (1 - kap)
    # not even the smallest
    assert np.all(4.0 * up.astype(np.float64) * margin * (1.0 - eps) > 4.0 * (n2 + e * (2 * n1 + e)) * (1.0 - 1e-7))
    low = f32(4.0) * r2 * (f32(1.0) - kap)
    assert np.all(low.astype(np.float64) * (1.0 + eps) <= 4.0 * (n2 - 2 * e * n1) * (1.0 + 1e-7))


def test_the_clip_uses_these_windows():
    src = (Path(__file__).resolve().parent.parent / "paper_2412_04514_amd" / "csrc" / "clip.hip").read_text()
    src = src.replace("__builtin_amdgcn_sqrtf", "sqrt")
    for form in ("nv = sqrt(d2) * sqrt(R2up)", "((float)a.eps + 5e-7f) * c + (wv + 5e-7f) * nv",
                 "(float)a.eps * (c + nv) * (1.0f + 1e-4f)",
                 "(wv + 2e-6f) * (c + sqrt(2.0f * c) * sqrt(R2up))",
                 "(3.5f + verrel) * verrel + 2.0f * (float)a.eps + 4e-6f",
                 "fmaxf(16.0f * (float)a.eps, FLT_EPSILON)", "(float)a.eps + 1.7321f * verrel"):
        assert form in src, form


# The stream phase's boxes and balls, in the clip's precision: a box that holds a
# point of a vertex' ball meets it, and a point that cuts a vertex off may cut.
def box_meets(lo, hi, v, r, t):
    g = np.maximum(t(0), np.maximum(lo - v, v - hi))
    return (g[:, 0] * g[:, 0] + g[:, 1] * g[:, 1]) + g[:, 2] * g[:, 2] <= r * r


@pytest.mark.parametrize("scale", [1e-14, 1e-10, 1e-5, 1.0])
@pytest.mark.parametrize("t", [np.float32, np.float64])
def test_boxes_that_hold_a_point_of_a_ball_meet_it(scale, t):
    rng = np.random.default_rng(13)
    n = 200_000
    v = (rng.standard_normal((n, 3)) * scale).astype(t)
    e = (np.abs(v).max(axis=1) * 10.0 ** rng.uniform(-8, -4.8, n)).astype(f32) if t is np.float32 else np.zeros(n)
    norm = np.sqrt((v[:, 0] * v[:, 0] + v[:, 1] * v[:, 1]) + v[:, 2] * v[:, 2], dtype=t)
    rad = norm * t(1.0 + 1e-5) + t(4.0) * e
    # a centre within the error bounds, and a point on its ball's surface
    c = v.astype(np.float64) + rng.choice([-1.0, 1.0], (n, 3)) * e[:, None].astype(np.float64)
    q = rng.standard_normal((n, 3))
    q = c + q / np.linalg.norm(q, axis=1, keepdims=True) * np.linalg.norm(c, axis=1, keepdims=True)
    side = rng.uniform(0, 1, (2, n, 3)) * scale * 10.0 ** rng.uniform(-6, 0, (2, n, 1))
    lo, hi = q - side[0], q + side[1]
    if t is np.float32:  # rounded outward
        flo, fhi = lo.astype(f32), hi.astype(f32)
        lo = np.where(flo > lo, np.nextafter(flo, f32(-np.inf)), flo)
        hi = np.where(fhi < hi, np.nextafter(fhi, f32(np.inf)), fhi)
    assert np.all(box_meets(lo, hi, v, rad, t))


@pytest.mark.parametrize("R", [1e-14, 1e-10, 1e-8, 1e-2, 1.0])
@pytest.mark.parametrize("ratio", [1e-4, 1e-3, 1e-1, 1.9])
def test_points_that_cut_a_vertex_may_cut(R, ratio):
    # the double clip: n.v - c > 0 by as little as double tells
    rng = np.random.default_rng(14)
    u = rng.standard_normal((100_000, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    v = u * R
    a = rng.standard_normal(u.shape)
    a -= (a * u).sum(axis=1, keepdims=True) * u
    a /= np.linalg.norm(a, axis=1, keepdims=True)
    d = R * ratio
    along = 0.5 * d * d / R
    n = along * u + np.sqrt(max(d * d - along * along, 0.0)) * a
    c = 0.5 * ((n[:, 0] * n[:, 0] + n[:, 1] * n[:, 1]) + n[:, 2] * n[:, 2])
    over = (n.astype(np.longdouble) * v).sum(axis=1) - 0.5 * (n.astype(np.longdouble) ** 2).sum(axis=1)
    cuts = over > 0
    far = np.maximum((n[:, 0] * v[:, 0] + n[:, 1] * v[:, 1]) + n[:, 2] * v[:, 2], -c)
    w = 1e-12 * (c + np.abs(n).sum(axis=1) * np.sqrt((v * v).sum(axis=1)))
    assert cuts.sum() > 10_000 and not np.any(far[cuts] < (c - w)[cuts])
