"""GPU test of the plain pixel resolve: a wave takes 256 entries, 4 consecutive
pixels per lane where they are one aligned run of the output and each pixel by
itself elsewhere. The same images come out of the general resolve kernel (a
render that asks for the time of flight as well), bit for bit, at image sizes
whose tiles cross cameras, branches and cloaks, misaligned ones included."""
import pytest

from paper_1209_6038_amd import workloads as W
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("res,spp,n", [(1, 1, 1), (3, 1, 2), (15, 4, 2), (16, 1, 3), (16, 4, 1), (17, 1, 5),
                                       (18, 9, 2), (32, 4, 3), (34, 1, 2), (65, 4, 1), (64, 16, 1)])
def test_plain_resolve_equals_the_general_one(res, spp, n):
    import torch
    from paper_1209_6038_amd import rt
    cl = [rt.Cloak(W.cloak(a, height=W.HEIGHT)) for a in (0, 1)]
    cams = W.orbit_frames(n, res, spp)
    say(f"case resolve tiles res={res} spp={spp} n={n}")
    plain = torch.full((2, n, 2, res, res, 3), -1.0, device="cuda")
    rt.render_multi(cl, W.render_opts(), W.room(), cams, 3, out=plain)
    general = torch.full((2, n, 2, res, res, 3), -1.0, device="cuda")
    rt.render_multi(cl, W.render_opts(), W.room(), cams, 3, out=general, aux=("tof",))
    torch.cuda.synchronize()
    assert torch.equal(plain, general)
    assert (plain >= 0).all()
