"""GPU: adaptive density control (Sec. 4.3) through the C ABI against the
oracle -- rotation and scale of the conditional covariance, and one clone /
split / prune step."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests import _gpu as G

pytestmark = pytest.mark.gpu


def _scene(n, seed):
    return synth.make_scene(synth.SceneSpec(n=n, seed=seed, l_cross_std=0.4))


def test_decompose_matches_oracle():
    from paper_2410_04974_amd import _lib
    pn = _scene(20000, 31)
    R, S = _lib.decompose(G.to_dev(pn))
    R = R.cpu().numpy().astype(np.float64).transpose(2, 0, 1)  # [n, 3, 3]
    S = S.cpu().numpy().astype(np.float64).T
    Ro, So = oracle.decompose(pn)
    assert np.abs(S - So).max() <= 2e-5 * So.max()
    sig = np.einsum("nij,nj,nkj->nik", Ro, So ** 2, Ro)
    rec = np.einsum("nij,nj,nkj->nik", R, S ** 2, R)
    scale = np.abs(sig).max(axis=(1, 2), keepdims=True)
    assert (np.abs(rec - sig) / scale).max() < 2e-5
    assert np.abs(np.einsum("nji,njk->nik", R, R) - np.eye(3)).max() < 2e-5
    assert np.abs(np.linalg.det(R) - 1.0).max() < 2e-5
    # the axes themselves are unique only with distinct scales; there the sign
    # convention makes them equal
    gap = np.minimum(So[:, 0] - So[:, 1], So[:, 1] - So[:, 2]) / So[:, 0]
    ok = gap > 2e-2
    print("decompose: S err", np.abs(S - So).max() / So.max(), "distinct-scale fraction", ok.mean(), flush=True)
    assert ok.mean() > 0.5
    assert np.abs(R[ok] - Ro[ok]).max() < 2e-3


def test_density_step_matches_oracle():
    from paper_2410_04974_amd import Renderer
    n = 4000
    pn = _scene(n, 37)
    rng = np.random.default_rng(38)
    pn[75] = rng.normal(0.0, 2.5, n).astype(np.float32)  # some opacities below 0.01
    # visible counts 0..3 and mean gradients far from the threshold 2e-4
    cnt = rng.integers(0, 4, n).astype(np.float32)
    avg = np.where(rng.random(n) < 0.5, 5e-4, 5e-5).astype(np.float32)
    stats = np.stack([avg * cnt, cnt]).astype(np.float32)
    _, So = oracle.decompose(pn)
    # put the clone / split size threshold in a gap of the largest scales
    smax = np.sort(So.max(axis=1))
    k = np.argmax(np.diff(smax[n // 3: 2 * n // 3])) + n // 3
    thr = 0.5 * (smax[k] + smax[k + 1])
    extent, pdense = 1.0, float(thr)
    d, margins = oracle.decisions(pn, stats, 2e-4, pdense, extent, 0.01)
    assert np.abs(margins).min() > 1e-4  # no decision within float32 reach (~1e-6) of its threshold
    assert set(np.unique(d)) == {0, 1, 2, 3}
    noise = rng.normal(size=(2, 3, n)).astype(np.float32)
    m = rng.normal(size=(76, n)).astype(np.float32)
    v = np.abs(rng.normal(size=(76, n))).astype(np.float32)
    lam = rng.normal(size=n).astype(np.float32)
    ref = oracle.densify(pn, stats, noise, 2e-4, pdense, extent, 0.01, m=m, v=v, lambda_raw=lam)
    r = Renderer()
    po, mo, vo, lo = r.ctx.densify(G.to_dev(pn), torch.from_numpy(stats).to(G.DEV),
                                   torch.from_numpy(noise).to(G.DEV), 2e-4, pdense, extent, 0.01,
                                   m=G.to_dev(m), v=G.to_dev(v), lambda_raw=torch.from_numpy(lam).to(G.DEV))
    po, mo, vo, lo = (t.cpu().numpy() for t in (po, mo, vo, lo))
    print("density step:", n, "->", po.shape[1], "decisions", np.bincount(d, minlength=4), flush=True)
    assert po.shape == ref["params"].shape
    assert np.array_equal(mo, ref["m"].astype(np.float32)) and np.array_equal(vo, ref["v"].astype(np.float32))
    assert np.array_equal(lo, ref["lambda_raw"].astype(np.float32))
    # kept and cloned Gaussians are bitwise copies; split children within float32 rounding of
    # mu_p + R (S z) (R, S from float32 Sigma_cond) and of the rescaled Cholesky rows
    sizes = np.array([0, 1, 2, 2])[d]
    parent = np.repeat(np.arange(n), sizes)
    split = np.repeat(d == 3, sizes)
    assert np.array_equal(po[:, ~split], pn[:, parent[~split]])
    diff = np.abs(po[:, split] - ref["params"][:, split])
    sc = So[parent[split]].max(axis=1)
    assert (diff[0:3] / sc).max() < 1e-3
    assert diff[6:].max() < 1e-4
    assert np.array_equal(po[3:6, split], pn[3:6, parent[split]])


def test_training_continues_after_densify():
    """Statistics from training steps drive one density step (its size equals
    the oracle's plan on the same statistics); training then continues on the
    new set, with a learnable lambda carried along."""
    import math
    from paper_2410_04974_amd import Renderer, Trainer
    w, pn = G.scene("c2", 20000)
    cam = synth.default_camera(200, 160)
    tgt = Renderer().forward(torch.from_numpy(synth.perturbed(pn)).to(G.DEV), [cam])
    lam = torch.full((pn.shape[1],), math.log(0.35 / 0.65), device=G.DEV)
    tr = Trainer(G.to_dev(pn), Renderer(), lambda_raw=lam)
    stats = torch.zeros((2, pn.shape[1]), device=G.DEV)
    for _ in range(5):
        tr.step([cam], tgt, densify=stats)
    torch.cuda.synchronize()
    p_before = tr.params.cpu().numpy()
    d, _ = oracle.decisions(p_before, stats.cpu().numpy(), 1e-5, 0.01, 2.0, 0.01)
    n_new = tr.densify(stats, extent=2.0, grad_threshold=1e-5)
    print("densify:", pn.shape[1], "->", n_new, "decisions", np.bincount(d, minlength=4), flush=True)
    assert n_new == int(np.array([0, 1, 2, 2])[d].sum())
    assert tr.lambda_raw.shape[0] == n_new and tr.m.shape[1] == n_new
    losses = [float(tr.step([cam], tgt)) for _ in range(3)]
    assert all(math.isfinite(x) for x in losses)


@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 700])
@pytest.mark.parametrize("kind", ["keep", "clone", "split", "mixed"])
@pytest.mark.parametrize("moments", [False, True])
def test_density_apply_block_edges(n, kind, moments):
    """The apply lists up to two outputs for each of 256 parents per workgroup:
    one Gaussian, whole and cut workgroups, no and only doubled outputs.
    Copies are bitwise, children within float32 rounding (as above)."""
    from paper_2410_04974_amd import Renderer
    pn = _scene(n, 41)
    rng = np.random.default_rng(42)
    pn[75] = 1.0
    grow = {"keep": np.zeros(n, bool), "clone": np.ones(n, bool), "split": np.ones(n, bool),
            "mixed": rng.random(n) < 0.6}[kind]
    if kind == "mixed":
        pn[75, rng.random(n) < 0.3] = -6.0
    stats = np.stack([np.where(grow, 5e-4, 5e-5), np.ones(n)]).astype(np.float32)
    _, So = oracle.decompose(pn)
    smax = np.sort(So.max(axis=1))
    pdense = {"keep": 1.0, "clone": 1e3, "split": 1e-6}.get(kind)
    if pdense is None:
        i = int(np.argmax(np.diff(smax))) if n > 1 else 0
        pdense = float(0.5 * (smax[i] + smax[min(i + 1, n - 1)])) if n > 1 else 1.0
    noise = rng.normal(size=(2, 3, n)).astype(np.float32)
    m, v = (rng.normal(size=(76, n)).astype(np.float32) for _ in range(2))
    d, _ = oracle.decisions(pn, stats, 2e-4, pdense, 1.0, 0.01)
    sizes = np.array([0, 1, 2, 2])[d]
    if sizes.sum() == 0:
        pytest.skip("every Gaussian pruned")
    ref = oracle.densify(pn, stats, noise, 2e-4, pdense, 1.0, 0.01, m=m, v=v)
    mom = dict(m=G.to_dev(m), v=G.to_dev(v)) if moments else {}
    po, mo, vo, _ = Renderer().ctx.densify(G.to_dev(pn), torch.from_numpy(stats).to(G.DEV),
                                           torch.from_numpy(noise).to(G.DEV), 2e-4, pdense, 1.0, 0.01, **mom)
    po = po.cpu().numpy()
    assert po.shape == ref["params"].shape
    if moments:
        assert np.array_equal(mo.cpu().numpy(), ref["m"].astype(np.float32))
        assert np.array_equal(vo.cpu().numpy(), ref["v"].astype(np.float32))
    parent, split = np.repeat(np.arange(n), sizes), np.repeat(d == 3, sizes)
    assert np.array_equal(po[:, ~split], pn[:, parent[~split]])
    if split.any():
        diff = np.abs(po[:, split] - ref["params"][:, split])
        assert (diff[0:3] / So[parent[split]].max(axis=1)).max() < 1e-3
        assert diff[6:].max() < 1e-4
        assert np.array_equal(po[3:6, split], pn[3:6, parent[split]])
