"""Payloads of 256 voxels a side and more, whose voxel index passes 2^24: the
forward and the payload gradient (closed-form runs and sample loop), FP32 and
BF16, one primitive and a few rays, against the FP64 oracle.

Tolerances.  A voxel coordinate u < 512 carries at most 2^-16 of rounding by
itself, and that of the local position y (|a| < 8: 2^-22, times (M-1)/2 < 160),
so 6e-5 on each axis; a sample's value is off by at most 3 times that of its
range, and opacity and premultiplied colour by at most twice that of 1 (largest
opacity over its mean): 4e-4.  A trilinear weight is off by at most 2e-4 and
is 0.19 in the root mean square: 1e-3 of the payload gradient.  (The position
gradient is not compared: too many samples lie within rounding of a voxel face
at this resolution.)"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_grads, max_abs, say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,steps,bf16", [(256, 64, True), (257, 64, False), (300, 64, False), (300, 2048, False), (300, 64, True)])
def test_index_past_24_bits(mvp_ctx, m, steps, bf16):
    prims = scenes.random_box_scene(701, n=1, m=2, s_lo=0.5, s_hi=0.6)
    rng = np.random.default_rng(702)
    prims.payload = rng.random((1, m, m, m, 4), dtype=np.float32)
    prims.pos[:] = 0
    if bf16:
        prims = scenes.as_bf16(prims)
    cam = scenes.look_at_camera(np.random.default_rng(703), 12, 10)
    params = scenes.MarchParams(1.0 / steps, 1e-6)
    dp = DevicePrims.from_host(prims, bf16=bf16)
    acc = mvp_ctx.build_accel(dp, [cam], params)
    rgba, aux = acc.render_fwd(dp)
    up = np.random.default_rng(704).normal(size=(cam.height * cam.width, 4))
    ref, gref = oracle.render_grad(prims, cam, params, up)
    err = max_abs(rgba.cpu().numpy().reshape(-1, 4), ref["rgba"])
    say(f"{m}^3, {steps} samples per unit, bf16 {bf16}: {int((ref['rgba'][:, 3] > 0).sum())} rays hit, max-abs {err:.2e}")
    assert (ref["margin"] >= 1e-3).all()
    assert err <= 4e-4
    g = acc.render_bwd(dp, aux, torch.from_numpy(up.astype(np.float32)).cuda().reshape(rgba.shape))
    torch.cuda.synchronize()
    check_grads({"payload": g["payload"].cpu().numpy()}, {"payload": gref["payload"]}, 1e-3, ("payload",))
    acc.destroy()
