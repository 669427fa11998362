"""GPU test of how a render's camera records reach the device: by value, 8 per
launch, for up to 64 cameras, as a copy beyond. Every camera's image must be
that of its own render, also when renders of other cameras are issued before
and after it on the same stream without waiting."""
import pytest

from paper_1209_6038_amd import workloads as W
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 8, 9, 64, 65])
def test_images_do_not_depend_on_the_number_of_cameras(n):
    import torch
    from paper_1209_6038_amd import rt
    cl = [rt.Cloak(W.cloak(0, height=W.HEIGHT))]
    cams = W.orbit_frames(n, 16, 1)  # one sample per pixel: jitter is keyed by the camera index
    assert len(cams) == n
    say(f"case camera records n={n}")
    one = [rt.render_multi(cl, W.render_opts(), W.room(), [c], 3) for c in cams[:3] + cams[-3:]]
    full = rt.render_multi(cl, W.render_opts(), W.room(), cams, 3)
    again = [rt.render_multi(cl, W.render_opts(), W.room(), [c], 3) for c in cams[:3] + cams[-3:]]
    torch.cuda.synchronize()
    for k, (a, b) in enumerate(zip(one, again)):
        i = k if k < len(cams[:3]) else n - len(cams[-3:]) + k - len(cams[:3])
        assert torch.equal(a[0, 0], full[0, i]) and torch.equal(b[0, 0], full[0, i]), i
    if n > 1:
        assert not torch.equal(full[0, 0], full[0, 1])
