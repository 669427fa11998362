"""GPU test of how rays are dealt to waves, for every scheme with and without the
Eq. (12) weights and every accepted block size: a ray's result is the same bits
whatever the launch's shape and whatever else is in it, up to more rays than the
chip's first round of waves takes."""
import pytest

from paper_1209_6038_amd import workloads as W
from tests.gpu_helpers import say
from tests.test_gpu_scheduling import _rays, _same

pytestmark = pytest.mark.gpu

OPTS = {"dp45": W.opts_dp45(), "rk4": W.opts_rk4(1e-2), "ham": W.opts_rk4_ham(2e-2),
        "hamc": W.opts_rk4_hamc(1e-2)}
SHAPES = [(64, 1), (128, 16), (192, 0), (192, 3), (256, 1024)]


@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("axis,branch", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("scheme", list(OPTS))
def test_rays_do_not_depend_on_the_launch(scheme, axis, branch, trans):
    import torch
    from paper_1209_6038_amd import rt
    cl = rt.Cloak(W.cloak(axis, height=W.HEIGHT))
    op = {**OPTS[scheme], "max_steps": 3000}  # near-axis rays run out of steps
    x = torch.from_numpy(_rays(200_003, 37)).cuda()
    full = rt.trace_batch(cl, op, branch, x, with_trans=trans)
    for n in (1, 65, 1025, 200_003):
        part = x if n == x.shape[1] else x[:, 7:7 + n].contiguous()
        at = 0 if n == x.shape[1] else 7
        for block, refill in [(0, 0)] + SHAPES:
            say(f"case launch {scheme} axis={axis} branch={branch} trans={trans} n={n} block={block} refill={refill}")
            got = rt.trace_batch(cl, {**op, "block": block, "refill_period": refill}, branch, part, with_trans=trans)
            torch.cuda.synchronize()
            for key in full:
                assert _same(got[key], full[key][..., at:at + n]), (key, n, block, refill)
    cl.close()


@pytest.mark.parametrize("scheme", list(OPTS))
def test_mixed_branches_do_not_depend_on_the_launch(scheme):
    """All four branches in one launch, against each branch on its own."""
    import torch
    from paper_1209_6038_amd import rt
    from paper_1209_6038_amd import surrogate as S
    cl = [rt.Cloak(W.cloak(a, height=W.HEIGHT)) for a in (W.RADIAL, W.AZIMUTHAL)]
    op = {**OPTS[scheme], "max_steps": 3000}
    x = S.features(120_001, 19)
    want = rt.transit_exact(cl, op, x, hres=True, nsteps=True)
    for block, refill in SHAPES:
        say(f"case mixed launch {scheme} block={block} refill={refill}")
        got = rt.transit_exact(cl, {**op, "block": block, "refill_period": refill}, x, hres=True, nsteps=True)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert _same(a, b), (block, refill)
    for k in range(4):
        sel = torch.nonzero((x[4] == (k & 1)) & (x[5] == (k >> 1))).flatten()
        got = rt.transit_exact(cl, op, x[:, sel].contiguous(), hres=True, nsteps=True)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert _same(a, b[..., sel]), k
    for c in cl:
        c.close()
