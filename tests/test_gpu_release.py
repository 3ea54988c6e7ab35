"""What a tessellation asks of the caller's allocator: memory goes back only when
nothing on the stream uses it any more (an allocator need not know about
streams), and cells built on the host need little beside the call's buffers."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

vt = pytest.importorskip("paper_2412_04514_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


class Watched(vt.Context):
    """Notes for each release whether the stream had work left, and the most
    bytes that were out at a time."""

    def __init__(self):
        super().__init__()
        self.busy, self.peak = [], 0
        alloc_ = self._alloc_cb

        def alloc(nbytes, user):
            p = alloc_(nbytes, user)
            self.peak = max(self.peak, sum(t.numel() for t in self._live.values()))
            return p

        def release(p, _user):
            self.busy.append(not torch.cuda.current_stream().query())
            self._live.pop(int(p or 0), None)

        self._inner = alloc_
        self._alloc_cb = vt._lib.ALLOC_FN(alloc)
        self._release_cb = vt._lib.RELEASE_FN(release)
        self.lib.votess_set_allocator(self.handle, self._alloc_cb, self._release_cb, None)


def _shell(m, n, seed):
    # a cell of m faces, more than the fast kernels hold, among n others
    rng = np.random.default_rng(seed)
    u = rng.standard_normal((m, 3))
    shell = 0.5 + 0.1 * u / np.linalg.norm(u, axis=1, keepdims=True) + 1e-4 * rng.standard_normal(u.shape)
    bg = rng.random((n, 3))
    return np.concatenate([[[0.5, 0.5, 0.5]], shell, bg[np.linalg.norm(bg - 0.5, axis=1) > 0.25]])


@pytest.mark.parametrize("kw", [dict(k0=64, max_gpu_retries=1), dict(k0=64, max_gpu_retries=0), dict(k0=32),
                                dict(k0=0), dict(k0=32, faces=True, vertices=True),
                                dict(k0=32, force_fail_every=50)], ids=str)
@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_nothing_is_released_in_use(kw, dt):
    ctx = Watched()
    P = torch.from_numpy(_shell(60, 20_000, 3).astype(dt)).cuda()
    torch.cuda.synchronize()
    r = vt.tessellate(P, ctx=ctx, precision="f32" if dt is np.float32 else "f64", **kw)
    assert len(ctx.busy) > 5 and not any(ctx.busy)
    if kw.get("max_gpu_retries") == 1:
        assert r.stats["capacity_cells"] > 0  # with lists of its own


def test_nothing_is_released_in_use_after_an_error():
    ctx = Watched()
    P = torch.rand(20_000, 3, device="cuda")
    P[1] = P[0]
    with pytest.raises(vt.VotessError):
        vt.tessellate(P, ctx=ctx)
    with pytest.raises(vt.VotessError):
        vt.tessellate(torch.rand(20_000, 3, device="cuda") + 0.5, ctx=ctx)
    assert len(ctx.busy) > 5 and not any(ctx.busy)


@pytest.mark.parametrize("every", [1, 7])
@pytest.mark.parametrize("kw", [dict(), dict(vertices=True, faces=True)], ids=str)
def test_cells_built_on_the_host_need_little_memory(kw, every):
    P = torch.from_numpy(np.random.default_rng(4).random((20_000, 3))).cuda()
    a, b = Watched(), Watched()
    on_gpu = vt.tessellate(P, ctx=a, **kw)
    on_host = vt.tessellate(P, ctx=b, force_fail_every=every, **kw)
    assert on_host.stats["fallback_cells"] >= len(P) // every
    assert b.peak <= a.peak + (16 << 20)
    # every row in its place, whatever chunk it came in
    assert torch.equal(on_gpu.row_ptr, on_host.row_ptr) and torch.equal(on_gpu.col, on_host.col)
    assert torch.all((on_gpu.volume - on_host.volume).abs() <= 2e-12 * on_gpu.volume)
    if kw:
        assert torch.equal(on_gpu.vrow_ptr, on_host.vrow_ptr)
        assert torch.all((on_gpu.centroid - on_host.centroid).abs() <= 1e-9)
        # (areas of tiny faces: relative to the cell's largest)
        assert torch.all((on_gpu.area - on_host.area).abs() <= 1e-9 * on_gpu.area.max())
