"""The backward of payloads whose gradient does not fit the LDS, taken in slabs
of cell layers (17^3 to 45^3) or in device memory (larger): rays along and
across the slabs and parallel to them, both ways through a pair, items full of
pairs, saturating rays whose clamping sample falls in some slab.  Against the
FP64 oracle with the gradients' gates.  The upstream gradient is zero on rays
whose stop the oracle's margin calls close, and on rays with a sample within
rounding of a voxel face, where the position derivative of the trilinear field
jumps and the cell a sample belongs to is a matter of rounding."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import GROUPS, check_grads, say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu

# name: (primitives, payload size, opacity factor, width, samples per unit, combine, viewing axis or None)
CASES = {
    "17-two-slabs": (3, 17, 2.0, 20, 256, "sum", None),
    "24-sequential": (3, 24, 6.0, 18, 256, "sequential", None),
    "32-along-z": (2, 32, 1.0, 15, 512, "sum", 2),
    "32-parallel-to-slabs": (2, 32, 1.0, 15, 512, "sum", 0),
    "32-short-runs": (2, 32, 4.0, 16, 64, "sum", None),
    "45-slabs-of-one-layer": (1, 45, 2.0, 14, 512, "sum", None),
    "46-device-memory": (1, 46, 2.0, 14, 512, "sum", None),
}


def near_a_face(prims, cam, params):
    """Rays with a sample closer than 3e-6 M voxels (FP32 rounding of the voxel
    coordinate is about 2e-7 M) to a face between two cells."""
    m, dt = prims.m, params.step
    px, py = np.meshgrid(np.arange(cam.width) + 0.5, np.arange(cam.height) + 0.5)
    d = np.stack([px, py, np.ones_like(px)], -1).reshape(-1, 3) @ cam.pix2dir.astype(np.float64).T
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    near = np.zeros(len(d), bool)
    for k in range(prims.n):
        A = prims.rot[k].astype(np.float64).T / prims.scale[k].astype(np.float64)[:, None]
        a, b = A @ (cam.origin.astype(np.float64) - prims.pos[k]), d @ A.T
        tau = np.arange(int(6.0 / dt)) * dt
        u = (a[None, None, :] + tau[None, :, None] * b[:, None, :] + 1) * 0.5 * (m - 1)
        inside = ((u >= 0) & (u <= m - 1)).all(-1)
        face = np.rint(u)
        close = (np.abs(u - face) < 3e-6 * m) & (face > 0) & (face < m - 1)
        near |= (close.any(-1) & inside).any(-1)
    return near


@pytest.mark.parametrize("name", list(CASES))
def test_backward_slabs(mvp_ctx, name):
    n, m, opac, width, steps, combine, axis = CASES[name]
    prims = scenes.random_box_scene(501, n=n, m=m, s_lo=0.4, s_hi=0.7)
    prims.pos *= np.float32(0.4)
    prims.payload[..., 3] *= np.float32(opac)
    cam = scenes.look_at_camera(np.random.default_rng(502), width, width)
    if axis is not None:
        prims.rot[:] = np.eye(3, dtype=np.float32)
        origin = np.zeros(3)
        origin[axis] = 3.0
        cam = scenes.axis_camera(width, width, origin, forward_axis=axis)
    params = scenes.MarchParams(1.0 / steps, 1e-6, combine=combine)
    dp = DevicePrims.from_host(prims)
    acc = mvp_ctx.build_accel(dp, [cam], params)
    rgba, aux = acc.render_fwd(dp)
    ref = oracle.render(prims, cam, params)
    up = np.random.default_rng(503).normal(size=ref["rgba"].shape)
    up[ref["margin"] < 1e-4] = 0
    if axis is None:   # (an axis-parallel ray keeps to one cell per axis)
        up[near_a_face(prims, cam, params)] = 0
    assert (np.abs(up).sum(1)[ref["rgba"][:, 3] > 0] > 0).sum() >= 12
    say(f"{name}: {int((ref['rgba'][:, 3] > 0).sum())} covered rays, {int((ref['rgba'][:, 3] >= 1).sum())} saturated")
    _, gref = oracle.render_grad(prims, cam, params, up)
    g = acc.render_bwd(dp, aux, torch.from_numpy(up.astype(np.float32)).cuda().reshape(rgba.shape))
    torch.cuda.synchronize()
    check_grads({k: g[k].cpu().numpy() for k in GROUPS}, gref, 1e-4, GROUPS, floor=0.1)
    acc.destroy()


def test_items_full_of_pairs(mvp_ctx):
    """One 32^3 box over all of a 96 x 96 picture: an item of 16 tiles of 256 rays,
    every ray a pair; the gradient of the summed opacity."""
    prims = scenes.random_box_scene(504, n=1, m=32, s_lo=0.9, s_hi=1.0)
    prims.pos[:] = 0
    prims.payload[..., 3] *= np.float32(0.02)
    cam = scenes.look_at_camera(np.random.default_rng(505), 96, 96)
    cam.pix2dir[:, :2] *= np.float32(0.4)
    fwd = -cam.origin / np.linalg.norm(cam.origin)
    cam.pix2dir[:, 2] = fwd - cam.pix2dir[:, :2] @ np.float32([48, 48])
    params = scenes.MarchParams(1.0 / 64, 1e-6)
    dp = DevicePrims.from_host(prims)
    acc = mvp_ctx.build_accel(dp, [cam], params)
    rgba, aux = acc.render_fwd(dp)
    assert int((rgba[..., 3] > 0).sum()) > 8000
    up = np.zeros((96 * 96, 4))
    up[:, 3] = 1.0
    up[near_a_face(prims, cam, params)] = 0
    _, gref = oracle.render_grad(prims, cam, params, up)
    g = acc.render_bwd(dp, aux, torch.from_numpy(up.astype(np.float32)).cuda().reshape(rgba.shape))
    torch.cuda.synchronize()
    check_grads({k: g[k].cpu().numpy() for k in GROUPS}, gref, 1e-4, GROUPS, floor=0.1)
    acc.destroy()
