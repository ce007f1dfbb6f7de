"""The forward's walk in each of its forms -- keeping the backward's state with
few and with many tiles, image only, counting contributors -- over short lists
and lists past its steps and chunks, pixels that stop, alpha above its clamp and
blocks cut by the image's edge.  The images lie in the oracle's decision
envelope, and the forms agree bitwise."""
import numpy as np
import pytest

import oracle
import synth
from tests import _gpu as G
from tests.test_gpu_backward_walk import stack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opacity", ["faint", "dense", "clamped"])
@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 127, 129, 300])
def test_forward_forms_match_envelope_and_each_other(n, opacity):
    from paper_2410_04974_amd import _lib
    p = stack(n, opacity)
    cam = synth.default_camera(37, 21)
    bg = (0.3, 0.1, 0.2)
    r, pt, imgs = G.render(p, [cam], bg=bg)
    T, last = r.ctx.export(_lib.EXPORT_T_FINAL), r.ctx.export(_lib.EXPORT_LAST)
    env = oracle.render_envelope(p, cam, oracle.Settings(bg=bg))
    G.check_envelope(imgs[0], T.reshape(cam.height, cam.width), env, f"{n} {opacity}",
                     lambda *a: print(*a, flush=True))
    cached = r.forward_cached(pt, _lib.build_cache(pt), [cam])[0].cpu().numpy()
    assert np.array_equal(cached, imgs[0])
    rc, _, counted = G.render(p, [cam], bg=bg, flags=_lib.FLAG_COUNTS)
    assert np.array_equal(counted[0], imgs[0])
    assert np.array_equal(rc.ctx.export(_lib.EXPORT_T_FINAL), T)
    assert np.array_equal(rc.ctx.export(_lib.EXPORT_LAST), last)
    cnt = rc.ctx.export(_lib.EXPORT_COUNTS).reshape(cam.height, cam.width)
    ok = ~env["ambiguous"]
    assert np.array_equal(cnt[ok], env["ncontrib"][ok])


@pytest.mark.parametrize("opacity", ["dense", "clamped"])
def test_forward_many_tiles_equals_single_views(opacity):
    """Sixteen 512x512 views make 16,384 tiles, where the forward takes its form
    for many; a view on its own takes the one for few."""
    from paper_2410_04974_amd import _lib
    p = stack(700, opacity)
    cams = synth.fibonacci_cameras(16, [(512, 512)])
    r, pt, batch = G.render(p, cams, chunk=128)
    T = r.ctx.export(_lib.EXPORT_T_FINAL).reshape(16, -1)
    for k in (0, 5, 15):
        r1, _, one = G.render(p, [cams[k]], chunk=128)
        assert np.array_equal(one[0], batch[k])
        assert np.array_equal(r1.ctx.export(_lib.EXPORT_T_FINAL), T[k])
