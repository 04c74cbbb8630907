"""A structure built from primitives of one payload size and rendered with
another (the payload may differ from the build's): the backward's work items were
cut for the build's size, from the 128 entries of sparse rays over small
payloads to the 16 of large ones.  Pictures equal those of a structure
built with the payload they are rendered with, bit for bit; gradients are the
same sums over other work items: a few hundred FP32 additions per pose value,
5e-5 of the largest."""
import numpy as np
import pytest
import torch

from gpu_util import GROUPS, say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu


# payload sizes of the build and of the render; 40 samples per unit are 3 per cell of 8^3, under 3 of 16^3
@pytest.mark.parametrize("built,m", [(8, 4), (8, 16), (8, 20), (8, 46), (4, 12), (16, 8), (32, 8), (20, 16), (46, 24)])
@pytest.mark.parametrize("combine", ["sum", "sequential"])
def test_backward_with_another_payload_size(mvp_ctx, built, m, combine):
    width = 320
    prims = scenes.random_box_scene(801, n=5, m=m, s_lo=0.6, s_hi=0.9)
    prims.pos *= np.float32(0.2)
    cam = scenes.look_at_camera(np.random.default_rng(802), width, width)
    params = scenes.MarchParams(1.0 / 40, 1e-6, combine=combine)
    rays = torch.from_numpy(np.random.default_rng(803).choice(width * width, 800, replace=False)).cuda()
    dp = DevicePrims.from_host(prims)
    other = DevicePrims(dp.pos, dp.rot, dp.scale, torch.ones((5, built, built, built, 4), device="cuda"))
    up = torch.randn((800, 4), generator=torch.Generator("cuda").manual_seed(804), device="cuda")
    got = []
    for p in (other, dp):
        acc = mvp_ctx.build_accel(p, [cam], params, rays=rays)
        rgba, aux = acc.render_fwd(dp)
        got.append((rgba, acc.render_bwd(dp, aux, up)))
        say(f"built with {p.m}^3: {acc.info()['n_tile_pairs']} entries, loads {acc.load_counts()}")
        acc.destroy()
    (rgba, g), (rgba0, g0) = got
    assert torch.equal(rgba, rgba0) and float(rgba0[:, 3].max()) > 0.5
    for k in GROUPS:
        a, b = g[k].double(), g0[k].double()
        assert float((a - b).abs().max()) <= 5e-5 * float(b.abs().max()), k
