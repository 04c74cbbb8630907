"""Rounding of the offsets that the backward's closed-form runs work with.  A
44^3 payload under rays that are farther apart than its cells, several samples
to a run, so that a voxel's gradient comes from one run or two and a run's
offset error is not averaged away.  The upstream gradient is that of the summed
opacity: a voxel's opacity gradient is a sum of trilinear weights times dt.

With y rounded to 2^-25 / sqrt(3) at most in the root mean square (|y| < 1) and
the offset formed from it with one more rounding, an offset is off by 1.7e-8 times
(M-1)/2 = 3.7e-7, a weight (three offsets of 0.58 each, rms) by 1.1e-6 of
itself; rounding the whole coordinate (up to 43: 1.1e-6 rms above 32, half of
that above 16) first would give 2.1e-6."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import rel_l2, say
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [1101, 1102, 1103])
def test_weights_of_a_run(mvp_ctx, seed):
    prims = scenes.random_box_scene(seed, n=1, m=44, s_lo=0.7, s_hi=0.8)
    prims.pos[:] = 0
    prims.payload[..., 3] *= np.float32(0.01)
    cam = scenes.look_at_camera(np.random.default_rng(seed), 32, 32)
    params = scenes.MarchParams(1.0 / 256, 1e-6)
    dp = DevicePrims.from_host(prims)
    acc = mvp_ctx.build_accel(dp, [cam], params)
    rgba, aux = acc.render_fwd(dp)
    up = np.zeros((32 * 32, 4))
    up[:, 3] = 1.0
    _, gref = oracle.render_grad(prims, cam, params, up)
    g = acc.render_bwd(dp, aux, torch.from_numpy(up.astype(np.float32)).cuda().reshape(rgba.shape))
    lc = acc.load_counts()
    acc.destroy()
    e = rel_l2(g["payload"].cpu().numpy()[..., 3], gref["payload"][..., 3])
    say(f"{lc['prim_samples'] / lc['bwd_cell_runs']:.1f} samples per run, rel-L2 {e:.2e}")
    assert e <= 1.4e-6


@pytest.mark.parametrize("steps", [257, 300, 574])
def test_weights_at_rounded_sample_times(mvp_ctx, steps):
    """The same where dt is no power of two, so that the sample times fl(j dt) are not
    equidistant: near tau = 3 they are off by 0.7e-7 in the root mean square, which
    is 2e-6 of a voxel here and 6e-6 of a weight if a run takes them as equidistant.
    To first order (a tenth of it left) 0.6e-6, with the 1.1e-6 above 1.3e-6; gate
    1.8e-6."""
    prims = scenes.random_box_scene(1111, n=1, m=44, s_lo=0.7, s_hi=0.8)
    prims.pos[:] = 0
    prims.payload[..., 3] *= np.float32(0.01)
    cam = scenes.look_at_camera(np.random.default_rng(1111), 32, 32)
    params = scenes.MarchParams(1.0 / steps, 1e-6)
    dp = DevicePrims.from_host(prims)
    acc = mvp_ctx.build_accel(dp, [cam], params)
    rgba, aux = acc.render_fwd(dp)
    up = np.zeros((32 * 32, 4))
    up[:, 3] = 1.0
    _, gref = oracle.render_grad(prims, cam, params, up)
    g = acc.render_bwd(dp, aux, torch.from_numpy(up.astype(np.float32)).cuda().reshape(rgba.shape))
    acc.destroy()
    e = rel_l2(g["payload"].cpu().numpy()[..., 3], gref["payload"][..., 3])
    say(f"{steps} samples per unit, rel-L2 {e:.2e}")
    assert e <= 1.8e-6
