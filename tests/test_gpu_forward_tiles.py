"""GPU test of the fused inference at the edges of its tiles (128 rows, worked
on as two halves of 64): an entry's targets are the same bits whatever batch it
is in, and the reference's within the tolerance of the forward test."""
import numpy as np
import pytest

from oracle import mlp
from tests.gpu_helpers import say
from tests.test_gpu_surrogate import _oracle_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 63, 64, 65, 127, 128, 129, 300])
def test_forward_at_tile_edges(n):
    import torch
    from paper_1209_6038_amd import rt
    m = rt.Surrogate(seed=3)
    x = np.random.default_rng(1).normal(size=(6, 1500)).astype(np.float32)
    full = m.forward(torch.from_numpy(x).cuda())
    say(f"case forward tiles n={n}")
    first = m.forward(torch.from_numpy(x[:, :n].copy()).cuda())
    last = m.forward(torch.from_numpy(x[:, 1500 - n:].copy()).cuda())
    torch.cuda.synchronize()
    assert torch.equal(first, full[:, :n]) and torch.equal(last, full[:, 1500 - n:])
    ref, _ = mlp.forward(_oracle_params(m.get_params()), mlp.features(x[:, :n]), bf16=True)
    assert np.abs(first.cpu().numpy().T - ref).max() <= 2e-5
