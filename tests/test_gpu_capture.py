"""A structure whose first forward and backward are captured into a HIP graph:
what those calls make once per structure (the per-ray pairs, the lists of the
backward) has to be there for calls outside the graph, before and between its
replays, and for every replay.  Structures whose lists take the caller's stream,
the second stream (more than 32768 entries) and whose pairs are left to the first
forward, against the same calls without a graph: pictures bit for bit, gradients to 1e-6 of
the largest (only the order of the FP32 atomics between work items differs)."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_util import GROUPS, say
from paper_2103_01954_amd import _lib as L
from paper_2103_01954_amd import scenes
from paper_2103_01954_amd.api import DevicePrims, _stream

pytestmark = pytest.mark.gpu


def _zeros(dp):
    return {"payload": torch.zeros(dp.payload.shape, device="cuda"), "pos": torch.zeros_like(dp.pos),
            "rot": torch.zeros_like(dp.rot), "scale": torch.zeros_like(dp.scale)}


def _backward(ctx, acc, dp, aux, up, g):
    for v in g.values():
        v.zero_()
    cp = dp.c_struct()
    L.check("mvp_render_bwd_noalloc", ctx.lib.mvp_render_bwd_noalloc(
        ctx.handle, acc.handle, C.byref(cp), aux.data_ptr(), up.data_ptr(), *[g[k].data_ptr() for k in GROUPS], _stream()))


def _same(got, want, what):
    for k in GROUPS:
        d, m = float((got[k] - want[k]).abs().max()), float(want[k].abs().max())
        assert m > 0 and d <= 1e-6 * m, (what, k, d, m)


# primitives, payload size, width, half extents, MVP_PAIRS_IN_FORWARD
@pytest.mark.parametrize("n,m,width,s,pairs_in_forward", [
    (8, 8, 64, 0.3, "0"), (8, 8, 64, 0.3, "1"), (256, 8, 512, 0.5, "0"), (256, 6, 512, 0.5, "1"), (9000, 4, 128, 0.05, "0")])
@pytest.mark.parametrize("forward_captured", [True, False])
def test_first_calls_captured(mvp_ctx, monkeypatch, n, m, width, s, pairs_in_forward, forward_captured):
    monkeypatch.setenv("MVP_PAIRS_IN_FORWARD", pairs_in_forward)
    prims = scenes.random_box_scene(901, n=n, m=m, s_lo=s, s_hi=1.1 * s)
    prims.payload[..., 3] *= np.float32(min(1.0, 16.0 / n))
    cam = scenes.look_at_camera(np.random.default_rng(902), width, width)
    params = scenes.MarchParams(1.0 / 64, 1e-6)
    dp = DevicePrims.from_host(prims)
    gen = torch.Generator("cuda").manual_seed(903)
    up = torch.randn((1, width, width, 4), generator=gen, device="cuda")
    payloads = [torch.rand(dp.payload.shape, generator=gen, device="cuda") * min(1.0, 16.0 / n) for _ in range(3)]

    def eager(acc):
        rgba, aux = acc.render_fwd(dp)
        g = _zeros(dp)
        _backward(mvp_ctx, acc, dp, aux, up, g)
        return rgba, aux, g

    ref = mvp_ctx.build_accel(dp, [cam], params)
    want0 = eager(ref)
    acc = mvp_ctx.build_accel(dp, [cam], params)
    say(f"{n} of {m}^3: {acc.info()}")
    assert n != 256 or acc.info()["n_tile_pairs"] > 32768
    rgba, aux, g = torch.zeros_like(want0[0]), want0[1].clone(), _zeros(dp)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        if forward_captured:
            acc.render_fwd(dp, rgba=rgba, aux=aux)
        _backward(mvp_ctx, acc, dp, aux, up, g)
    got = eager(acc)       # before any replay
    assert torch.equal(got[0], want0[0])
    _same(got[2], want0[2], "eager before a replay")
    assert acc.info()["n_ray_pairs"] == ref.info()["n_ray_pairs"] > 0
    for i, pay in enumerate(payloads):
        dp.payload.copy_(pay)
        want = eager(ref)
        if not forward_captured:
            aux.copy_(want[1])
        graph.replay()
        torch.cuda.synchronize()
        if forward_captured:
            assert torch.equal(rgba, want[0]), i
        _same(g, want[2], f"replay {i}")
        assert acc.load_counts()["bwd_pairs_replayed"] == ref.load_counts()["bwd_pairs_replayed"] > 0
        between = eager(acc)
        _same(between[2], want[2], f"eager after replay {i}")
    acc.destroy()
    ref.destroy()
