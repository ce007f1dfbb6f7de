"""The calls that wait for their stream: the growing forward's pair count and
the density plan's output count, also when the stream is busy for far longer
than the host watches for the count itself (2 ms)."""
import ctypes
import time

import numpy as np
import pytest
import torch

import synth
from tests import _gpu as G

pytestmark = pytest.mark.gpu


def keep_busy(ms=25.0):
    """Work of a good ms milliseconds on the current stream; returns its inputs (to be held)."""
    a = torch.ones((4096, 4096), device=G.DEV)
    out = torch.empty_like(a)
    torch.mm(a, a, out=out)
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    torch.mm(a, a, out=out)
    end.record()
    end.synchronize()
    for _ in range(int(ms / start.elapsed_time(end)) + 1):
        torch.mm(a, a, out=out)
    return a, out


def plan_call(ctx, params, stats):
    """sixdgs_densify_plan as a call without arguments, and its count."""
    from paper_2410_04974_amd import _lib as L
    d = L.DensitySettings(2e-4, 0.01, 4.0, 0.01)
    n_out = ctypes.c_int64(-1)
    args = (ctx._h, ctypes.c_void_p(params.data_ptr()), params.shape[1], ctypes.c_void_p(stats.data_ptr()),
            ctypes.byref(d), ctypes.byref(n_out), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    f = L.lib().sixdgs_densify_plan
    return (lambda: f(*args)), n_out


def density_inputs(n):
    pn = synth.make_scene(synth.SceneSpec(n=n, seed=3))
    rng = np.random.default_rng(4)
    cnt = rng.integers(0, 4, n).astype(np.float32)
    stats = np.stack([np.where(rng.random(n) < 0.5, 5e-4, 5e-5).astype(np.float32) * cnt, cnt])
    return G.to_dev(pn), torch.from_numpy(stats).to(G.DEV)


def test_growing_forward_behind_long_work():
    w, pn = G.scene("c2", 30000)
    p, cam = G.to_dev(pn), synth.default_camera(400, 300)
    want = G.renderer().forward(p, [cam])[0].clone()
    r = G.renderer()
    r.forward(p, [synth.default_camera(32, 32)])  # the pair buffers have to grow behind the work
    torch.cuda.synchronize()
    held = keep_busy()
    t = time.perf_counter()
    img = r.forward(p, [cam])[0]
    waited = time.perf_counter() - t
    torch.cuda.synchronize()
    print(f"waited {1e3 * waited:.1f} ms", flush=True)
    assert waited > 5e-3
    assert torch.equal(img, want)
    r.ctx.check()
    del held


def test_density_plan_behind_long_work():
    params, stats = density_inputs(50000)
    r = G.renderer()
    call, n_out = plan_call(r.ctx, params, stats)
    assert call() == 0
    want = n_out.value
    held = keep_busy()
    n_out.value = -1
    t = time.perf_counter()
    assert call() == 0
    waited = time.perf_counter() - t
    print(f"waited {1e3 * waited:.1f} ms, {n_out.value} outputs", flush=True)
    assert waited > 5e-3 and n_out.value == want
    del held


def test_density_plan_leaves_its_stream_idle():
    """The plan is done when the call returns (its offsets may be read on any
    stream), not only its count."""
    params, stats = density_inputs(300000)
    hip = ctypes.CDLL("libamdhip64.so")
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            r = G.renderer()
            call, _ = plan_call(r.ctx, params, stats)
            handle = ctypes.c_void_p(stream.cuda_stream)
            torch.cuda.synchronize()
            query = hip.hipStreamQuery
            states = []
            for _ in range(200):
                rc = call()
                states.append((rc, query(handle)))
            torch.cuda.synchronize()
        print("busy on return:", sum(q != 0 for _, q in states), "of", len(states), flush=True)
        assert states == [(0, 0)] * 200
