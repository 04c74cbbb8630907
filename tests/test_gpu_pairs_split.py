"""The pairs of a ray subset's tiles on both sides of the line between one lane
per entry and one lane per ray (a quarter of the list's length per block of 64
entries): pictures and pair counts equal the full image's exactly."""
import numpy as np
import pytest
import torch

from gpu_util import say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu


# primitives (all of them in most tiles' lists) and rays in each tile of 16 x 16 pixels
@pytest.mark.parametrize("n,rays_per_tile", [(3, 1), (4, 1), (20, 5), (20, 6), (64, 16), (64, 17), (65, 8), (65, 9), (128, 16),
                                             (128, 17), (129, 16)])
def test_lane_per_entry_and_per_ray(mvp_ctx, n, rays_per_tile):
    prims = scenes.random_box_scene(1501, n=n, m=4, s_lo=0.6, s_hi=1.0)
    prims.payload[..., 3] *= np.float32(2.0 / n)
    cam = scenes.look_at_camera(np.random.default_rng(1502), 48, 32)
    params = scenes.MarchParams(1.0 / 64, 1e-6)
    rng = np.random.default_rng(1503)
    pix = np.arange(48 * 32)
    tile = (pix // 48 // 16) * 3 + (pix % 48) // 16
    ids = np.concatenate([rng.permutation(pix[tile == k])[:rays_per_tile] for k in range(6)])
    ids = torch.from_numpy(rng.permutation(ids).astype(np.int64)).cuda()
    dp = DevicePrims.from_host(prims)
    full = mvp_ctx.build_accel(dp, [cam], params)
    sub = mvp_ctx.build_accel(dp, [cam], params, rays=ids)
    want, aux = full.render_fwd(dp)
    got, sub_aux = sub.render_fwd(dp)
    assert torch.equal(got, want.reshape(-1, 4)[ids])
    assert torch.equal(sub_aux, aux.reshape(-1)[ids])
    off, _ = full.debug_hits(dp)
    hits = int((off[1:] - off[:-1])[ids.cpu().numpy()].sum())
    pairs = sub.info()["n_ray_pairs"]
    say(f"{n} primitives, {rays_per_tile} rays a tile: {pairs} pairs of {hits} hits")
    assert 0 < pairs <= hits
    full.destroy()
    sub.destroy()
