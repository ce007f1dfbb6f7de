"""The compositing backward's screen-space gradients (of each Gaussian's mean,
conic, opacity and colour on the image) for long thin Gaussians,
against float64 sums over the very records the kernels read."""
import ctypes

import numpy as np
import pytest
import torch

import synth
from tests import _gpu as G
from tests.test_gpu_backward_walk import stack

pytestmark = pytest.mark.gpu
F32 = np.float32
LOG2E = F32(1.4426950408889634)


def needles(length, n=40):
    """n faint Gaussians, exp(length) long in the world, a hundredth of that or
    a pixel wide, at all angles to the image's axes."""
    p = stack(n, "faint", seed=9)
    rng = np.random.default_rng(3)
    for k, v in zip(synth.DIAG_SPATIAL, (length, -4.0, -4.0)):
        p[synth.ROW_L + k] = v
    for i in (1, 2):  # the long axis' other two components
        p[synth.ROW_L + synth.tri_index(i, 0)] = rng.uniform(-2.0, 2.0, n)
    return p


def screen_gradients(r, n):
    """[n, 9] out of the workspace of a debug-mode context: du, dv, dQxx, dQxy, dQyy, dalpha, dr, dg, db."""
    from paper_2410_04974_amd import _lib as L
    ptr, nbytes = ctypes.c_void_p(), ctypes.c_int64()
    assert L.lib().sixdgs_debug_buffer(r.ctx._h, b"screen-space gradients", ctypes.byref(ptr),
                                       ctypes.byref(nbytes)) == L.OK
    out = np.empty((n, 9), np.float32)
    assert nbytes.value >= out.nbytes
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipMemcpy(ctypes.c_void_p(out.ctypes.data), ptr, ctypes.c_size_t(out.nbytes), 2) == 0
    return out.astype(np.float64)


def reference(rec, tiles, dl, bg=0.0):
    """The same in float64 with the covariance in the conic's place, each sum's
    absolute value, and the conic's: the exponent as the kernels round it (so
    that alpha is theirs), everything after it in 64 bits.  Also the pixels where
    a decision is near enough to go either way."""
    H, W = dl.shape[1:]
    fy, fx = [a.astype(F32) + F32(0.5) for a in np.mgrid[0:H, 0:W]]
    ids = [e for e in np.argsort(rec[:, G.REC_DEPTH], kind="stable") if tiles[e] > 0]
    taken = []
    T = np.ones((H, W))
    unsure = np.zeros((H, W), bool)
    for e in ids:
        u, v, qxx, qxy, qyy, ac = rec[e, :6].astype(F32)
        cA, cB, cC = F32(-0.5) * LOG2E * qxx, -LOG2E * qxy, F32(-0.5) * LOG2E * qyy
        dx, dy = fx - u, fy - v
        fma = lambda a, b, c: (a.astype(np.float64) * b + c).astype(F32)  # noqa: E731
        t = fma(dx, np.float64(cA), (cB * dy).astype(np.float64))
        p = fma(t, dx.astype(np.float64), fma((cC * dy).astype(F32), dy.astype(np.float64), np.float64(np.log2(ac))))
        p = p.astype(np.float64)
        unsure |= np.abs(p - np.log2(1 / 255)) < 1e-4
        a = np.where(p >= np.log2(1 / 255), np.exp2(p), 0.0)
        taken.append((e, a, T.copy(), (float(cA), float(cB) / 2, float(cC)), float(u), float(v)))
        T = T * (1 - a)
    unsure |= T < 0.02  # (a pixel may stop below 1e-2)
    dC = np.where(unsure, 0.0, dl.astype(np.float64))
    X, Y = np.arange(W)[None, :] + 0.5, np.arange(H)[:, None] + 0.5
    g, size, conic = np.zeros((len(rec), 9)), np.zeros((len(rec), 9)), np.zeros((len(rec), 2, 2))
    D = T * bg * dC.sum(0)  # dL/dC . the colour behind
    ln2 = np.log(2.0)
    for e, a, Tf, (cA, hB, cC), u, v in reversed(taken):
        c = rec[e, G.REC_R:G.REC_B + 1].astype(np.float64)
        dc = np.tensordot(c, dC, 1)
        w = Tf * a * dc - a / (1 - a) * D
        D = D + Tf * a * dc
        dx, dy = X - u, Y - v
        f0, f1 = cA * dx + hB * dy, hB * dx + cC * dy
        terms = [-2 * ln2 * w * f0, -2 * ln2 * w * f1, 2 * ln2**2 * w * f0 * f0, 2 * ln2**2 * w * f0 * f1,
                 2 * ln2**2 * w * f1 * f1, w / rec[e, G.REC_AC]] + [Tf * a * dC[k] for k in range(3)]
        g[e] = [t.sum() for t in terms]
        size[e] = [np.abs(t).sum() for t in terms]
        conic[e] = [[np.abs(0.5 * w * a * b).sum() for b in (dx, dy)] for a in (dx, dy)]
    return g, size, conic, unsure


def symmetric(a):
    return np.stack([np.stack([a[:, 0], a[:, 1]], -1), np.stack([a[:, 1], a[:, 2]], -1)], -2)


@pytest.mark.parametrize("length", [-1.0, 0.0, 1.0, 2.0])
@pytest.mark.parametrize("batch,chunk,tile", [(0, 0, (16, 16)), (256, 512, (32, 8))])
def test_needles_against_sums_in_64_bits(length, batch, chunk, tile):
    """Mean, opacity and colour within 2e-6 of the sum of their terms' absolute
    values (transmittance and colour behind take 40 roundings).  The conic's sums
    are float32, and the covariance's -Q G Q magnifies their rounding: the bound
    is eight roundings, 2^-24 each of the conic's absolute sums, magnified alike,
    and nowhere more than 1e-4 of the covariance's own absolute sums."""
    from paper_2410_04974_amd import _lib as L
    p = needles(length)
    n = p.shape[1]
    cam = synth.default_camera(301, 203)
    r, pt, _ = G.render(p, [cam], flags=L.FLAG_DEBUG, batch=batch, chunk=chunk, tile=tile)
    rec, tiles = G.records(r)
    dl = synth.upstream_gradient([cam])[0]
    ref, size, conic, unsure = reference(rec, tiles, dl)
    r.backward(pt, [torch.from_numpy(np.where(unsure, 0, dl).astype(np.float32)).to(G.DEV)])
    g = screen_gradients(r, n)
    Q = symmetric(rec[:, G.REC_QXX:G.REC_QYY + 1].astype(np.float64))
    cov = -(Q @ symmetric(g[:, 2:5]) @ Q)
    bound = 2e-6 * size
    for k, (i, j) in zip((2, 3, 4), ((0, 0), (0, 1), (1, 1))):
        g[:, k] = cov[:, i, j]
        magnified = (np.abs(Q) @ conic @ np.abs(Q))[:, i, j]
        bound[:, k] = np.minimum(bound[:, k] + 8 * 2.0**-24 * magnified, 1e-4 * size[:, k])
    seen = (tiles > 0) & (size.max(1) > 0)
    q = rec[seen].astype(np.float64)
    thin = 1 - q[:, G.REC_QXY] ** 2 / (q[:, G.REC_QXX] * q[:, G.REC_QYY])
    off = np.abs(g - ref)[seen]
    rel, of_bound = off / np.maximum(size[seen], 1e-30), off / np.maximum(bound[seen], 1e-30)
    print(length, batch, "Gaussians", int(seen.sum()), "1 - rho^2 at least", f"{thin.min():.1e} median {np.median(thin):.1e}",
          "kept", f"{1 - unsure.mean():.2f}", "off by at most", " ".join(f"{x:.1e}" for x in rel.max(0)),
          "of the bound", " ".join(f"{x:.2f}" for x in of_bound.max(0)), flush=True)
    assert seen.sum() >= 30 and unsure.mean() < 0.5
    assert of_bound.max() <= 1
