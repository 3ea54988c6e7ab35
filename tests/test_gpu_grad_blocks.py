"""Gradient of the list-size network over numbers of 64-sample blocks around
the 16 partial sums that the reduction loads at a time."""
import numpy as np
import pytest
import torch

from oracle import mlp

pytestmark = pytest.mark.gpu

pytest.importorskip("paper_2412_04514_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _model():
    from paper_2412_04514_amd import kmodel
    rng = np.random.default_rng(21)
    theta = (mlp.init_params(21) + rng.normal(scale=0.02, size=mlp.NPARAM)).astype(np.float32)
    mean, std = rng.normal(size=12), rng.uniform(0.5, 2.0, size=12)
    m = kmodel.KModel(seed=21)
    m.set_params(theta, mean, std)
    return m, theta.astype(np.float64), mean.astype(np.float32).astype(np.float64), \
        std.astype(np.float32).astype(np.float64)


def _batch(nb):
    rng = np.random.default_rng(22)
    return (rng.normal(size=(nb, 12)) * 1.5 + 0.5).astype(np.float32), rng.integers(0, 7, nb).astype(np.uint8)


def _grad(m, x, y):
    g, loss = m.grad(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    return g.cpu().numpy(), loss.cpu().numpy().reshape(())


@pytest.mark.parametrize("blocks", [2, 16, 32, 64])
def test_partials_are_added_in_order(blocks):
    # copies of one block have partials of its gradient / blocks, exactly, the
    # number being a power of two; their sum in order is then known bit for bit
    m, *_ = _model()
    x, y = _batch(64)
    one, loss = _grad(m, x, y)
    got, got_loss = _grad(m, np.tile(x, (blocks, 1)), np.tile(y, blocks))
    want, want_loss = np.zeros_like(one), np.float32(0)
    for _ in range(blocks):
        want = want + one / np.float32(blocks)
        want_loss = want_loss + loss / np.float32(blocks)
    np.testing.assert_array_equal(got, want)
    assert got_loss == want_loss


@pytest.mark.parametrize("nb", [64 * 15, 64 * 16 + 1, 64 * 31 + 63])
def test_sizes_around_the_unrolled_sum(nb):
    # FP32 sums and BF16 roundings that flip by one ulp in few of the samples:
    # the bounds that larger batches are held to
    m, theta, mean, std = _model()
    x, y = _batch(nb)
    g, loss = _grad(m, x, y)
    lref, gref = mlp.loss_and_grad(theta, x.astype(np.float64), y, mean, std, bf16_points=True)
    assert np.linalg.norm(g - gref) <= 1e-3 * np.linalg.norm(gref)
    assert abs(loss - lref) <= 1e-4 * abs(lref)
    step_loss = m.train_step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), lr=1e-3)
    if step_loss is not None:
        assert float(step_loss) == float(loss)
