"""The backward's two ways through a (ray, primitive) pair: cell runs in closed
form and the sample loop, on both sides of the rules that choose between them
and where a run has edges: rays parallel to the voxel axes (a zero slope),
runs longer than one part (64 samples), runs of one sample, a clamping sample
alone in its run, the sequential rule, the fade window, BF16.  Against the FP64
oracle with the gradients' gates (check_grads at 1e-4); upstream gradients on
rays whose stop the oracle's margin calls close are zero."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import GROUPS, check_grads, say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu

# name: (primitives, payload size, half extents, opacity factor, width, samples per unit, options, axis-parallel, spread)
CASES = {
    "axis-parallel": (4, 6, (0.3, 0.6), 1.0, 9, 128, {}, True, 1.0),
    "runs-of-many-parts": (5, 2, (0.3, 0.8), 0.05, 12, 2048, {}, False, 1.0),
    "three-samples-per-cell": (8, 8, (0.2, 0.3), 1.0, 20, 54, {}, False, 1.0),
    "under-three-samples": (8, 8, (0.2, 0.3), 1.0, 20, 40, {}, False, 1.0),
    "saturating-sequential": (8, 8, (0.2, 0.5), 20.0, 20, 128, {"combine": "sequential"}, False, 1.0),
    "saturating-sum": (8, 5, (0.3, 0.5), 40.0, 20, 64, {}, False, 1.0),
    "fade-bf16": (6, 8, (0.3, 0.6), 2.0, 16, 128, {"fade_alpha": 8.0, "bf16": True}, False, 1.0),
    "small-boxes-sample-loop": (12, 4, (0.03, 0.032), 20.0, 24, 512, {}, False, 0.08),
    "payload-in-device-memory": (3, 20, (0.3, 0.6), 1.0, 14, 256, {}, False, 1.0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_backward_runs(mvp_ctx, name):
    n, m, (lo, hi), opac, width, steps, opt, axis, spread = CASES[name]
    bf16 = bool(opt.get("bf16"))
    prims = scenes.random_box_scene(401, n=n, m=m, s_lo=lo, s_hi=hi)
    prims.pos *= np.float32(spread)
    prims.payload[..., 3] *= np.float32(opac)
    if bf16:
        prims = scenes.as_bf16(prims)
    cam = scenes.look_at_camera(np.random.default_rng(402), width, width)
    if spread < 1:   # a narrow view of the cluster
        cam.pix2dir[:, :2] *= np.float32(0.1)
        fwd = -cam.origin / np.linalg.norm(cam.origin)
        cam.pix2dir[:, 2] = fwd - cam.pix2dir[:, :2] @ np.float32([0.5 * width, 0.5 * width])
    if axis:
        prims.rot[:] = np.eye(3, dtype=np.float32)
        prims.pos[:, :2] *= np.float32(0.1)
        cam = scenes.axis_camera(width, width, (0.0, 0.0, 3.0))
    params = scenes.MarchParams(1.0 / steps, 1e-6, fade_alpha=opt.get("fade_alpha", 0.0),
                                combine=opt.get("combine", "sum"))
    dp = DevicePrims.from_host(prims, bf16=bf16)
    acc = mvp_ctx.build_accel(dp, [cam], params)
    rgba, aux = acc.render_fwd(dp)
    ref = oracle.render(prims, cam, params)
    up = np.random.default_rng(403).normal(size=ref["rgba"].shape)
    up[ref["margin"] < 1e-4] = 0
    say(f"{name}: {int((np.abs(up).sum(1) > 0).sum())} rays with an upstream gradient, "
        f"{int((ref['rgba'][:, 3] >= 1).sum())} saturated")
    _, gref = oracle.render_grad(prims, cam, params, up)
    g = acc.render_bwd(dp, aux, torch.from_numpy(up.astype(np.float32)).cuda().reshape(rgba.shape))
    torch.cuda.synchronize()
    check_grads({k: g[k].cpu().numpy() for k in GROUPS}, gref, 1e-4, GROUPS, floor=0.1)
    acc.destroy()
