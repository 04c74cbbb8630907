"""Payloads taken in slabs with values that fixed point cannot hold: a NaN or an
infinity in one box reaches the gradients of the voxels its rays touch and no
others, and a colour near the largest float leaves the other boxes' gradients
finite, as FP32 sums do.  Two boxes that share no ray; the second one's gradients
equal those without the odd value (the same pairs in another order and another
accumulator: 5e-5 of the largest)."""
import numpy as np
import pytest
import torch

from gpu_util import say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu


# payload size, boxes around the second (many items: the lists of the split), odd value, channel
@pytest.mark.parametrize("m,more", [(24, 0), (32, 700)])
@pytest.mark.parametrize("value,channel", [(np.nan, 3), (np.nan, 0), (np.inf, 1), (3e38, 2)])
def test_odd_values_stay_with_their_rays(mvp_ctx, m, more, value, channel):
    rng = np.random.default_rng(1801)
    prims = scenes.random_box_scene(1802, n=2 + more, m=m, s_lo=0.12, s_hi=0.2)
    prims.payload[..., 3] *= np.float32(0.2)
    cam = scenes.axis_camera(160, 96, (0.0, 0.0, 3.0))
    prims.pos[:] = np.array([0.6, 0.0, 0.0], np.float32) + rng.uniform(-0.2, 0.2, prims.pos.shape).astype(np.float32)
    prims.pos[0] = [-0.8, 0.0, 0.0]
    params = scenes.MarchParams(1.0 / 256, 1e-6)
    grads = []
    for odd in (False, True):
        if odd:
            prims.payload[0, 4:7, 5:8, 6:9, channel] = value
        dp = DevicePrims.from_host(prims)
        acc = mvp_ctx.build_accel(dp, [cam], params)
        rgba, aux = acc.render_fwd(dp)
        up = torch.randn(rgba.shape, generator=torch.Generator("cuda").manual_seed(1803), device="cuda")
        grads.append({k: v.cpu() for k, v in acc.render_bwd(dp, aux, up).items()})
        acc.destroy()
    ref, got = grads
    bad = int((~torch.isfinite(got["payload"][0])).sum())
    say(f"{m}^3, {value} in channel {channel}: {bad} of {got['payload'][0].numel()} values not finite")
    if np.isfinite(value):
        assert bool(torch.isfinite(got["payload"][1:]).all())
    else:
        assert 0 < bad < got["payload"][0].numel() // 2
    for k in ref:
        a, b = got[k][1:].double(), ref[k][1:].double()
        assert float((a - b).abs().max()) <= 5e-5 * float(b.abs().max()), k
