"""GPU test of rays whose step budget ends on the very step that brings them to
an internal reflection: they are out of steps inside the cloak like any other
such ray, without a residual at an exit."""
import numpy as np
import pytest

from paper_1209_6038_amd import workloads as W
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu

TIR, MAXSTEPS = 5, 3


@pytest.mark.parametrize("scheme", ["dp45", "rk4", "ham", "hamc"])
def test_budget_spent_at_an_internal_reflection(scheme):
    import torch
    from paper_1209_6038_amd import rt
    from paper_1209_6038_amd import surrogate as S
    op = {"dp45": W.opts_dp45(1e-8, r_out=W.R2), "rk4": W.opts_rk4(1e-2), "ham": W.opts_rk4_ham(2e-2),
          "hamc": W.opts_rk4_hamc(1e-2)}[scheme]
    cl = [rt.Cloak(W.cloak(a, height=W.HEIGHT)) for a in (W.RADIAL, W.AZIMUTHAL)]
    x = S.features(4000, 5)
    # no reflection allowed: a ray ends at its first one, with the steps it took to it
    _, st0, ns0 = rt.transit_exact(cl, {**op, "max_bounces": 0, "max_steps": 60}, x, nsteps=True)
    torch.cuda.synchronize()
    hit = 0
    for k in np.unique(ns0[st0 == TIR].cpu().numpy()):
        say(f"case step budget {scheme} max_steps={k}")
        at = (st0 == TIR) & (ns0 == int(k))
        y, st, hr, ns = rt.transit_exact(cl, {**op, "max_steps": int(k)}, x, hres=True, nsteps=True)
        torch.cuda.synchronize()
        assert (st[at] == MAXSTEPS).all() and (ns[at] == int(k)).all()
        assert torch.isnan(y[:, at]).all()
        assert torch.isnan(hr[st == MAXSTEPS]).all(), int(k)
        hit += int(at.sum())
    assert hit > 0
    for c in cl:
        c.close()
