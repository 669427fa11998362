"""GPU test that a batch's gradient does not see the workspace's earlier
contents: the weight gradients sum rows in whole steps of 64, and the rows past
a ragged batch's end hold what a larger batch left there."""
import numpy as np
import pytest

from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


def _batch(n, seed, scale=1.0):
    import torch
    r = np.random.default_rng(seed)
    return (torch.from_numpy(r.normal(size=(6, n)).astype(np.float32)).cuda(),
            torch.from_numpy((scale * r.normal(size=(5, n))).astype(np.float32)).cuda())


@pytest.mark.parametrize("n", [1, 15, 17, 63, 65, 127, 129, 385, 1000, 4095])
def test_smaller_batch_after_a_larger_one(n):
    """The same ragged batch after 4096 rows of large gradients and after 4096
    rows without weight (all dz zero): the same bits."""
    import torch
    from paper_1209_6038_amd import rt
    say(f"case gradient workspace n={n}")
    x0, t0 = _batch(4096, 1, 1e4)
    x, t = _batch(n, 2)
    got = []
    for w0 in (None, torch.zeros(4096, device="cuda")):
        m = rt.Surrogate(seed=8)
        m.grad(x0, t0, w0)
        got.append(m.grad(x, t))
        torch.cuda.synchronize()
        m.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
