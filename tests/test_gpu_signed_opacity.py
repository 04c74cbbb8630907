"""Payloads that are not physical opacities.  Negative densities, where a ray's
opacity falls again within the window of samples in which it crossed the limit:
against the FP64 oracle, which takes sample after sample, within the
forward's 1e-5 times the largest sums (densities of both signs up to 8, over
steps of 1/16: 4e-5).  The sequential rule on one box, where a sample has one
primitive (a sample of several is taken one by one only if its sum
saturates)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import max_abs, say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("combine,n,size", [("sum", 10, 0.4), ("sum", 1, 0.9), ("sequential", 1, 0.9)])
def test_negative_opacity(mvp_ctx, combine, n, size):
    prims = scenes.random_box_scene(1001, n=n, m=6, s_lo=0.9 * size, s_hi=1.1 * size)
    if n == 1:
        prims.pos[:] = 0
    prims.payload[..., 3] = np.random.default_rng(1002).uniform(-4, 8, prims.payload.shape[:-1]).astype(np.float32)
    cam = scenes.look_at_camera(np.random.default_rng(1003), 40, 30)
    params = scenes.MarchParams(1.0 / 16, 1e-6, combine=combine)
    dp = DevicePrims.from_host(prims)
    acc = mvp_ctx.build_accel(dp, [cam], params)
    rgba, aux = acc.render_fwd(dp)
    rs, ps = acc.counts()
    acc.destroy()
    ref = oracle.render(prims, cam, params)
    sure = ref["margin"] >= 1e-4
    stopped = sure & (ref["rgba"][:, 3] >= 1)
    say(f"{combine}: {int(stopped.sum())} stopped rays, {int(sure.sum())} sure")
    assert stopped.sum() > 100
    got = rgba.cpu().numpy().reshape(-1, 4).astype(np.float64)
    assert max_abs(got[sure], ref["rgba"][sure]) <= 4e-5
    if sure.all():
        assert rs == ref["ray_samples"].sum() and ps == ref["prim_samples"].sum()



def test_nan_opacity(mvp_ctx):
    """A NaN density makes a ray's colour NaN, under both combine rules alike."""
    prims = scenes.random_box_scene(1011, n=8, m=6, s_lo=0.3, s_hi=0.6)
    prims.payload[..., 3] *= np.float32(0.5)
    prims.payload[2, 2:4, 2:4, 2:4, 3] = np.nan
    cam = scenes.look_at_camera(np.random.default_rng(1012), 40, 30)
    dp = DevicePrims.from_host(prims)
    nan = {}
    for combine in ("sum", "sequential"):
        acc = mvp_ctx.build_accel(dp, [cam], scenes.MarchParams(1.0 / 64, 1e-6, combine=combine))
        nan[combine] = torch.isnan(acc.render_fwd(dp)[0])
        acc.destroy()
    say(f"{int(nan['sum'].any(-1).sum())} rays with a NaN")
    assert int(nan["sum"][..., :3].any(-1).sum()) > 5
    assert torch.equal(nan["sum"], nan["sequential"])
