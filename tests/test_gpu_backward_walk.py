"""The backward's walk over a tile's list, at the list lengths where it changes
form: groups of 16 Gaussians (one short, whole, one over), batches and chunks,
pixels that stop inside a group, alpha above its clamp, and blocks cut by the
image's edge -- against the FP64 oracle.  The bars are those of the other
gradient comparisons: 1e-3 relative per parameter group, and per element
1e-3 of max(|g|, 1e-2 max |g|)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests import _gpu as G
from tests.test_gpu_parity import _element_errors, _group_errors

pytestmark = pytest.mark.gpu

# raw opacity (mean, spread): faint Gaussians never saturate a pixel; dense
# ones stop it; in "clamped" every third has opacity 0.999
LOGITS = {"faint": (-3.0, 0.5), "dense": (-0.5, 0.5), "clamped": (-1.0, 0.5)}


def stack(n, opacity, seed=5):
    """n wide Gaussians around the origin: each covers most of a small image."""
    spec = synth.SceneSpec(n=n, means="cube", l_spatial_diag=(-1.0, 0.3), logit=LOGITS[opacity], seed=seed)
    p = synth.make_scene(spec)
    p[synth.ROW_MU_P:synth.ROW_MU_P + 3] *= 0.4
    c = synth.default_camera(8, 8).center
    p[synth.ROW_MU_D:synth.ROW_MU_D + 3] = (-c / np.linalg.norm(c))[:, None]  # seen along their own direction
    if opacity == "clamped":
        p[synth.ROW_OPACITY, ::3] = 7.0
    return p


def case(n, opacity, size):
    p = stack(n, opacity)
    cam = synth.default_camera(*size)
    env = oracle.render_envelope(p, cam)
    dl = synth.upstream_gradient([cam])[0].astype(np.float64)
    keep = ~G.grad_mask(env)
    dl[:, ~keep] = 0.0
    return p, cam, dl, float(keep.mean())


@pytest.mark.parametrize("opacity", ["faint", "dense", "clamped"])
@pytest.mark.parametrize("n,batch,chunk,tile", [
    (1, 0, 0, (16, 16)), (15, 0, 0, (16, 16)), (16, 0, 0, (32, 8)), (17, 64, 64, (16, 16)), (33, 0, 0, (8, 32)),
    (128, 0, 0, (16, 16)), (129, 128, 128, (16, 16)), (255, 256, 256, (16, 16)), (300, 256, 512, (32, 8)),
    (300, 64, 256, (16, 16)), (300, 0, 0, (16, 16))])
def test_backward_walk_forms(n, batch, chunk, tile, opacity):
    p, cam, dl, kept = case(n, opacity, (37, 21))
    r, pt, _ = G.render(p, [cam], batch=batch, chunk=chunk, tile=tile)
    g = r.backward(pt, [torch.from_numpy(dl.astype(np.float32)).to(G.DEV)]).cpu().numpy().astype(np.float64)
    ref, _ = oracle.backward(p, cam, dl)
    errs, el = _group_errors(g, ref), _element_errors(g, ref)
    print(n, opacity, "kept", f"{kept:.2f}", {k: f"{v:.1e}" for k, v in errs.items()},
          {k: f"{v:.2f}" for k, v in el.items()}, flush=True)
    assert kept > 0.3
    assert np.isfinite(g).all()
    assert all(v < 1e-3 for v in errs.values())
    assert all(v <= 1.0 for v in el.values())


@pytest.mark.parametrize("opacity", [0.5, 0.98])
def test_needles_stay_finite(opacity):
    """Gaussians so long and thin that the float32 exponent can come out above 0
    next to their axis: alpha stays below its clamp in both directions."""
    p = stack(40, "dense")
    for k, v in zip(synth.DIAG_SPATIAL, (3.5, -4.0, -4.0)):
        p[synth.ROW_L + k] = v + 0.01 * np.arange(40)
    p[synth.ROW_OPACITY] = np.log(opacity / (1 - opacity))
    cam = synth.default_camera(301, 203)
    r, pt, imgs = G.render(p, [cam])
    from paper_2410_04974_amd import _lib
    T = r.ctx.export(_lib.EXPORT_T_FINAL)
    rec, tiles = G.records(r)
    q = rec[tiles > 0]
    assert (q[:, G.REC_QXY] ** 2 > 0.999 * q[:, G.REC_QXX] * q[:, G.REC_QYY]).sum() >= 10
    g = r.backward(pt, [torch.from_numpy(synth.upstream_gradient([cam])[0]).to(G.DEV)])
    assert T.min() > 0 and T.max() <= 1 and np.isfinite(imgs[0]).all()
    assert torch.isfinite(g).all()
