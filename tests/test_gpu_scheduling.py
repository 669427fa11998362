"""GPU tests of how rays are dealt to waves: a ray's result is its own,
whatever else is in the launch. The integrator gives each wave its first rays
by number (one ray per wave for few rays, 64 and then chunks from the queue for
many), keeps the hardest rays' waves alone in a large segment, and shares the
waves out over the branches present, so every case is compared bit for bit with
the same rays in a launch of another shape, and the smaller one with the
oracle."""
import numpy as np
import pytest

import oracle
from paper_1209_6038_amd import workloads as W
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


def _same(a, b):
    import torch
    if a.dtype.is_floating_point:
        return torch.equal(torch.nan_to_num(a, nan=-7.0), torch.nan_to_num(b, nan=-7.0))
    return torch.equal(a, b)


def _rays(n, seed):
    """Random rays, every 64th aimed within 1e-2 .. 1e-4 of the axis (hundreds
    to thousands of attempts)."""
    x = W.random_rays(n, seed, z_range=(-1.0, 5.0))
    r = np.random.default_rng(seed + 1)
    k = np.arange(0, n, 64)
    a, p = r.uniform(0, 2 * np.pi, k.size), 10.0 ** r.uniform(-4, -2, k.size)
    x[0, k], x[1, k] = -p * np.sin(a) - 3 * np.cos(a), p * np.cos(a) - 3 * np.sin(a)
    x[3, k], x[4, k], x[5, k] = np.cos(a), np.sin(a), 0.0
    return x


@pytest.mark.parametrize("axis,branch", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_rays_do_not_depend_on_the_batch(axis, branch):
    import torch
    from paper_1209_6038_amd import rt
    cl = rt.Cloak(W.cloak(axis, height=W.HEIGHT))
    rays = _rays(200_003, 31)  # more entering rays than the chip's first round of waves takes
    x = torch.from_numpy(rays).cuda()
    full = rt.trace_batch(cl, W.opts_dp45(), branch, x)
    for n in (1, 63, 64, 65, 1023, 1025, 70_001):
        say(f"case scheduling axis={axis} branch={branch} n={n}")
        got = rt.trace_batch(cl, W.opts_dp45(), branch, x[:, 5:5 + n].contiguous())
        for block, refill in ((64, 1), (128, 16)):
            alt = rt.trace_batch(cl, W.opts_dp45(block=block, refill_period=refill), branch,
                                 x[:, 5:5 + n].contiguous())
            torch.cuda.synchronize()
            for key in full:
                assert _same(got[key], full[key][..., 5:5 + n]), (key, n)
                assert _same(got[key], alt[key]), (key, n, block)
    o = oracle.trace(W.cloak(axis, height=W.HEIGHT), W.opts_dp45(), branch, rays[:, :128])
    assert (full["status"][:128].cpu().numpy() == o["status"]).all()
    assert (full["nsteps"][:128].cpu().numpy() == o["nsteps"]).mean() > 0.95
    ok = np.isin(o["status"], (0, 1, 7)) & ~(o["hres"] > 1e-6)
    err = np.abs(full["out"][:, :128].cpu().numpy() - o["out"])[:, ok].max()
    assert err < 1e-6, err
    cl.close()


@pytest.mark.parametrize("counts", [(1, 0, 0, 1), (0, 0, 3000, 0), (300, 1, 120_000, 65), (90_000, 90_000, 1, 90_000)])
def test_branches_share_a_launch(counts):
    """Mixed launches of rt_transit_exact (radial o, e, azimuthal o, e) against
    each branch on its own."""
    import torch
    from paper_1209_6038_amd import rt
    say(f"case mixed counts={counts}")
    cl = [rt.Cloak(W.cloak(a)) for a in (W.RADIAL, W.AZIMUTHAL)]
    kind = np.repeat(np.arange(4), counts)
    x = W.surrogate_features(kind.size, 17)
    x[4], x[5] = kind & 1, kind >> 1
    perm = np.random.default_rng(3).permutation(kind.size)
    kind, x = kind[perm], torch.from_numpy(x[:, perm].copy()).cuda()
    op = W.opts_dp45(1e-8, r_out=W.R2)
    y, st, hr, ns = rt.transit_exact(cl, op, x, hres=True, nsteps=True)
    torch.cuda.synchronize()
    for k in range(4):
        sel = torch.from_numpy(np.flatnonzero(kind == k)).cuda()
        if sel.numel() == 0:
            continue
        y1, st1, hr1, ns1 = rt.transit_exact(cl, op, x[:, sel].contiguous(), hres=True, nsteps=True)
        torch.cuda.synchronize()
        assert _same(y[:, sel], y1) and _same(st[sel], st1) and _same(hr[sel], hr1) and _same(ns[sel], ns1), k
    for c in cl:
        c.close()
