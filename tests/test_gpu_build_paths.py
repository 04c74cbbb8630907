"""The build and the pairs kernel where a path ends: tiles with few rays for
their list (one lane per entry) and with more, lists about 64 and 128 entries
(one block, one staged chunk), rays parallel to the boxes' axes and through
their faces (the division without a shared reciprocal), more than 8192 tiles or
primitives (scans over several workgroups), a backward whose forward left no
state.  A subset's pictures equal the full image's bit for bit (the same pairs
and the same march); the others are held against the FP64 oracle within the
forward's 1e-5, counts exactly.  Gradients of the same pairs in another order:
at most a few hundred FP32 additions per pose value, 5e-5 of the largest."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import max_abs, oracle_pixels, say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu


def _gradients_close(got, want):
    for name in ("payload", "pos", "rot", "scale"):
        a, b = got[name].double(), want[name].double()
        assert float((a - b).abs().max()) <= 5e-5 * float(b.abs().max()), name


# primitives (all of them in most tiles' lists) and rays in each tile of 16 x 16 pixels
@pytest.mark.parametrize("n,rays_per_tile", [(1, 1), (20, 1), (20, 20), (20, 21), (64, 2), (65, 3), (128, 1), (128, 64),
                                             (128, 65), (129, 1), (200, 30), (200, 200), (20, 256)])
def test_subset_equals_full(mvp_ctx, n, rays_per_tile):
    prims = scenes.random_box_scene(401, n=n, m=4, s_lo=0.6, s_hi=1.0)
    prims.payload[..., 3] *= np.float32(2.0 / n)
    cam = scenes.look_at_camera(np.random.default_rng(402), 40, 32)
    params = scenes.MarchParams(1.0 / 64, 1e-6)
    rng = np.random.default_rng(403)
    pix = np.arange(40 * 32)
    tile = (pix // 40 // 16) * 3 + (pix % 40) // 16
    ids = np.concatenate([rng.permutation(pix[tile == k])[:rays_per_tile] for k in range(6)])
    ids = torch.from_numpy(rng.permutation(ids).astype(np.int64)).cuda()
    dp = DevicePrims.from_host(prims)
    full = mvp_ctx.build_accel(dp, [cam], params)
    sub = mvp_ctx.build_accel(dp, [cam], params, rays=ids)
    want, aux = full.render_fwd(dp)
    got, sub_aux = sub.render_fwd(dp)
    assert torch.equal(got, want.reshape(-1, 4)[ids])
    grad = torch.randn(got.shape, generator=torch.Generator("cuda").manual_seed(404), device="cuda")
    full_grad = torch.zeros_like(want)
    full_grad.reshape(-1, 4)[ids] = grad
    _gradients_close(sub.render_bwd(dp, sub_aux, grad), full.render_bwd(dp, aux, full_grad))
    full.destroy()
    sub.destroy()


@pytest.mark.parametrize("subset", [False, True])
def test_rays_along_axes_and_faces(mvp_ctx, subset):
    """Boxes along the world's axes; the middle column and row of pixels run
    parallel to them, one box has a face in the middle ray's plane and the
    camera lies in a box."""
    prims = scenes.random_box_scene(411, n=6, m=4, s_lo=0.2, s_hi=0.5)
    prims.rot[:] = np.eye(3, dtype=np.float32)
    prims.pos[:] = np.array([[0, 0, 0], [0.25, 0, 0.5], [0, -0.5, -0.5], [0.5, 0.5, 0], [0, 0, 2], [0, 3, 0]], np.float32)
    prims.scale[1:3] = 0.25
    prims.scale[2, 1] = 0.5
    prims.scale[4] = 0.5
    cam = scenes.axis_camera(33, 17, (0.0, 0.0, 2.0))
    params = scenes.MarchParams(1.0 / 64, 1e-6)
    ids = np.arange(33 * 17)[::7] if subset else None
    dp = DevicePrims.from_host(prims)
    acc = mvp_ctx.build_accel(dp, [cam], params, rays=None if ids is None else torch.from_numpy(ids).cuda())
    rgba, _ = acc.render_fwd(dp)
    off, hit = acc.debug_hits(dp)
    rs, ps = acc.counts()
    acc.destroy()
    pix = None if ids is None else oracle_pixels(cam, ids)
    ref = oracle.render(prims, cam, params, pixels=pix)
    want = oracle.hit_sets(prims, cam, params, pixels=pix)
    for r, w in enumerate(want):
        assert np.array_equal(hit[off[r]:off[r + 1]], w), r
    err = max_abs(rgba.cpu().numpy().reshape(-1, 4).astype(np.float64), ref["rgba"])
    say(f"axes, subset {subset}: max-abs {err:.2e}")
    assert err <= 1e-5
    if (ref["margin"] >= 1e-6).all():
        assert rs == ref["ray_samples"].sum() and ps == ref["prim_samples"].sum()


# name: primitives, half extents, image, samples per unit
BUILDS = {
    "8192-tiles": (30, (0.1, 0.3), (2048, 1024), 48),
    "more-tiles": (30, (0.1, 0.3), (2064, 1024), 48),
    "8191-primitives": (8191, (0.02, 0.05), (48, 33), 64),
    "8192-primitives": (8192, (0.02, 0.05), (48, 33), 64),
    "more-primitives": (9001, (0.02, 0.05), (48, 33), 64),
    "whole-image-rectangles": (70, (2.0, 3.0), (300, 200), 16),
}


@pytest.mark.parametrize("name", list(BUILDS))
def test_builds(mvp_ctx, name):
    n, (lo, hi), (width, height), steps = BUILDS[name]
    prims = scenes.random_box_scene(421, n=n, m=3, s_lo=lo, s_hi=hi)
    prims.payload[..., 3] *= np.float32(0.05)
    cam = scenes.look_at_camera(np.random.default_rng(422), width, height)
    params = scenes.MarchParams(1.0 / steps, 1e-6)
    ids = np.sort(np.random.default_rng(423).choice(width * height, 60, replace=False))
    dp = DevicePrims.from_host(prims)
    acc = mvp_ctx.build_accel(dp, [cam], params)
    rgba, _ = acc.render_fwd(dp, want_aux=False)     # no state for a backward
    again, aux = acc.render_fwd(dp)
    assert torch.equal(rgba, again)
    got = rgba.reshape(-1, 4)[torch.from_numpy(ids).cuda()].cpu().numpy().astype(np.float64)
    ref = oracle.render(prims, cam, params, pixels=oracle_pixels(cam, ids))
    err = max_abs(got, ref["rgba"])
    say(f"{name}: max-abs {err:.2e}")
    assert err <= 1e-5
    # the transposed lists: the gradient through the 60 rays, against a structure of those alone
    sub = mvp_ctx.build_accel(dp, [cam], params, rays=torch.from_numpy(ids).cuda())
    _, sub_aux = sub.render_fwd(dp)
    grad = torch.randn((60, 4), generator=torch.Generator("cuda").manual_seed(424), device="cuda")
    full_grad = torch.zeros_like(rgba)
    full_grad.reshape(-1, 4)[torch.from_numpy(ids).cuda()] = grad
    _gradients_close(acc.render_bwd(dp, aux, full_grad), sub.render_bwd(dp, sub_aux, grad))
    acc.destroy()
    sub.destroy()


# payload size, rays in each tile, rays in every 50th tile, dtype, fade: work items of
# sparse rays take 128 entries and 64 threads; 1024 pairs of one are ordered
@pytest.mark.parametrize("m,per_tile,crowd,bf16,fade", [(2, 1, 1, False, 0.0), (8, 1, 1, False, 0.0), (8, 6, 6, True, 0.0),
                                                        (10, 2, 200, False, 6.0), (8, 3, 250, True, 0.0),
                                                        (11, 1, 1, False, 0.0), (8, 9, 9, False, 0.0)])
def test_sparse_rays_backward(mvp_ctx, m, per_tile, crowd, bf16, fade):
    prims = scenes.random_box_scene(431, n=3, m=m, s_lo=1.0, s_hi=1.4, bf16=bf16)
    prims.payload[..., 3] *= np.float32(0.2)
    width, height = 400, 300
    cam = scenes.look_at_camera(np.random.default_rng(432), width, height)
    params = scenes.MarchParams(1.0 / 64, 1e-6, fade_alpha=fade, fade_beta=8.0 if fade else 0.0)
    rng = np.random.default_rng(433)
    pix = np.arange(width * height)
    tile = (pix // width // 16) * 25 + (pix % width) // 16
    ids = np.concatenate([rng.permutation(pix[tile == k])[:crowd if k % 50 == 0 else per_tile] for k in range(25 * 19)])
    ids = torch.from_numpy(ids.astype(np.int64)).cuda()
    dp = DevicePrims.from_host(prims)
    full = mvp_ctx.build_accel(dp, [cam], params)
    sub = mvp_ctx.build_accel(dp, [cam], params, rays=ids)
    want, aux = full.render_fwd(dp)
    got, sub_aux = sub.render_fwd(dp)
    assert torch.equal(got, want.reshape(-1, 4)[ids])
    grad = torch.randn(got.shape, generator=torch.Generator("cuda").manual_seed(434), device="cuda")
    full_grad = torch.zeros_like(want)
    full_grad.reshape(-1, 4)[ids] = grad
    _gradients_close(sub.render_bwd(dp, sub_aux, grad), full.render_bwd(dp, aux, full_grad))
    pose_only = {k: torch.zeros_like(getattr(dp, k)) for k in ("pos", "rot", "scale")}
    with_payload = sub.render_bwd(dp, sub_aux, grad)
    sub.render_bwd(dp, sub_aux, grad, pose_only)
    for k, v in pose_only.items():
        assert float((v - with_payload[k]).abs().max()) <= 5e-5 * float(v.abs().max()), k
    full.destroy()
    sub.destroy()
