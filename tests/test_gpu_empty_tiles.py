"""Pictures of which at least seven tiles in eight are empty: a wave of the march
then looks at several units together and writes the empty ones eight at a time.
Sizes that cut tiles and blocks, several views, no primitive at all, with and
without background and per-ray state; equal, bit for bit, to the same pixels as a
ray subset, which goes ray by ray."""
import numpy as np
import pytest
import torch

from gpu_util import say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu


# width, height, views, primitives, half extent
@pytest.mark.parametrize("width,height,views,n,size", [
    (700, 530, 1, 3, 0.02), (512, 512, 3, 6, 0.01), (2100, 1100, 1, 1, 0.3), (1500, 40, 2, 1, 0.01), (640, 640, 1, 0, 0.0),
    (513, 1025, 1, 40, 0.005)])
@pytest.mark.parametrize("background,state", [(False, True), (True, True), (True, False)])
def test_nearly_empty_pictures(mvp_ctx, width, height, views, n, size, background, state):
    prims = scenes.random_box_scene(1601, n=max(n, 1), m=4, s_lo=0.9 * size + 1e-3, s_hi=1.1 * size + 1e-3)
    prims.pos *= np.float32(0.3)
    prims = prims.subset(np.arange(n))
    rng = np.random.default_rng(1602)
    cams = [scenes.look_at_camera(rng, width, height) for _ in range(views)]
    params = scenes.MarchParams(1.0 / 512, 1e-6)
    dp = DevicePrims.from_host(prims)
    pix = views * width * height
    bg = torch.rand((pix, 3), generator=torch.Generator("cuda").manual_seed(1603), device="cuda") if background else None
    full = mvp_ctx.build_accel(dp, cams, params)
    sub = mvp_ctx.build_accel(dp, cams, params, rays=torch.arange(pix, device="cuda"))
    shape = (views, height, width)
    for _ in range(2):   # the second forward on the structure too
        got, aux = full.render_fwd(dp, rgba=torch.full(shape + (4,), 7.0, device="cuda"), want_aux=state,
                                   background=None if bg is None else bg.reshape(shape + (3,)))
        want, want_aux = sub.render_fwd(dp, want_aux=state, background=bg)
        assert torch.equal(got.reshape(-1, 4), want)
        if state:
            assert torch.equal(aux.reshape(-1), want_aux)
        assert full.counts() == sub.counts()
    tiles = views * ((width + 15) // 16) * ((height + 15) // 16)
    say(f"{tiles} tiles, {full.info()['n_tile_pairs']} entries, {full.counts()} samples")
    assert full.info()["n_tile_pairs"] * 8 <= tiles or n in (1, 40)
    full.destroy()
    sub.destroy()
