"""GPU test of the training kernels' tiling: the batch is cut into tiles of 16,
32 or 64 rows dealt to at most 256 blocks, and the weight gradients into up to
42 splits of whole 64-row steps, so the gradient is checked at the edges of
each: the smallest batches, one row more or less than a tile, the sizes where
the tile grows, more tiles than blocks (a ragged last one), a block's second
group of staged rows."""
import numpy as np
import pytest

from oracle import mlp
from tests.gpu_helpers import say
from tests.test_gpu_surrogate import _oracle_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65, 129, 4096, 4097, 8192, 8193, 16449, 40_001, 140_003])
def test_gradient_at_tile_edges(n):
    """Only some rows of a large batch carry weight, first, last and around
    the multiples of 16 and 64 among them: their gradient is the reference's
    over just those rows, within the bar of the gradient test at 300 rows
    (2^-3 of an entry's largest term for the BF16 roundings that fall the
    other way and 1e-4 of the summed magnitudes). The same batch twice gives
    the same bits, and NaN targets of rows without weight do not matter."""
    import torch
    from paper_1209_6038_amd import rt
    m = rt.Surrogate(seed=8)
    p = _oracle_params(m.get_params())
    rng = np.random.default_rng(n)
    x = rng.normal(size=(6, n)).astype(np.float32)
    t = rng.normal(size=(5, n)).astype(np.float32)
    rows = np.arange(n)
    if n > 300:
        rows = np.unique(np.concatenate([[0, 15, 16, 31, 32, 63, 64, n - 66, n - 65, n - 64, n - 17, n - 16, n - 2,
                                          n - 1], rng.choice(n, 250, replace=False)]))
    w = np.zeros(n, np.float32)
    w[rows] = 1.0
    t[:, w == 0.0] = np.nan
    args = [torch.from_numpy(a).cuda() for a in (x, t, w)]
    say(f"case training tiles n={n}")
    g, loss = m.grad(*args, huber=0.5)
    g2, loss2 = m.grad(*args, huber=0.5)
    torch.cuda.synchronize()
    assert torch.equal(g, g2) and torch.equal(loss, loss2)
    g = g.cpu().numpy().astype(np.float64)
    f, tt = mlp.features(x[:, rows]), t[:, rows].T.astype(np.float64)
    scale = len(rows) / n
    # the mean is over all n rows: the reference scales dy, not its result, so
    # that it rounds the same values to BF16
    lo, go = mlp.loss_and_grads(p, f, tt, w=np.full(5, scale), bf16=True, huber=0.5)
    assert abs(loss.item() - lo) <= 1e-5 * lo
    S, Mx = mlp.grad_term_magnitudes(p, f, tt, bf16=True, huber=0.5)
    off = 0
    for i, gg in enumerate(go):
        gpu = g[off:off + gg.size].reshape(gg.shape)
        bar = (1e-4 * S[i] + 2.0 ** -3 * Mx[i]) * scale
        assert (np.abs(gpu - gg) <= bar).all(), i
        off += gg.size
