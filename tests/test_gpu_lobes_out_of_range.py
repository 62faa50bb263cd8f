"""Spherical-Voronoi sums that leave [2^-100, 2^100], in which the unshifted lobes
are evaluated again with shifted logits: sites whose sums overflow, whose sums all
but vanish, and ordinary ones beside them, in one face.  That they do leave the
range for rendered rays is asserted.  Raster, walk and both backward passes against
the float64 oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from conftest import assert_grad_close
from test_gpu_modes import PARAMS, _grads

pytestmark = pytest.mark.gpu


def _case(kind):
    sc = W.scene_uniform(60, seed=4)
    sc.radius = (sc.radius * 2.0).astype(np.float32)
    cams = [W.pinhole(e, 11, 9, 55.0) for e in W.random_eyes(2, 2.7, 8)]
    rng = np.random.default_rng(1)
    sc.tex = np.array(sc.tex)
    axes = sc.tex[:, :, 3:27].reshape(60, 8, 8, 3)
    view = -np.asarray(cams[0].c2w)[:, 2]
    if kind in ("large", "all"):
        axes[:, :3] = 150.0 * rng.normal(size=(60, 3, 8, 3))
    if kind in ("vanishing", "all"):
        axes[:, 3:5] = 160.0 * view + 5.0 * rng.normal(size=(60, 2, 8, 3))
    sc.tex[:, :, 3:27] = axes.reshape(60, 8, 24)
    return sc, cams


@pytest.mark.parametrize("kind", ["large", "vanishing", "all"])
@pytest.mark.parametrize("walk", [False, True])
def test_matches_oracle(kind, walk):
    import paper_2604_24994_amd as pf
    print(f"case sums out of range: {kind}, walk {walk}", flush=True)
    sc, cams = _case(kind)
    d = oracle.generate_rays(cams[0])[1].numpy()
    axes = sc.tex[:, :, 3:27].reshape(-1, 8, 3).astype(np.float64)
    s2 = np.einsum("kma,ra->rkm", axes, d) / np.log(2.0)
    top = s2.max(-1) + np.log2(np.exp2(s2 - s2.max(-1, keepdims=True)).sum(-1))
    large, small = (top > 100).any(0).reshape(60, 8), (top < -100).any(0).reshape(60, 8)
    assert (large.any(1).mean() > 0.9) == (kind != "vanishing")
    assert (small[:, 3:5].mean() > 0.9) == (kind != "large")
    assert not (large | small)[:, 5:].any()
    rng = np.random.default_rng(7)
    Gs = [rng.normal(size=(c.n_rays, 4)) for c in cams]
    g, imgs = _grads(pf, sc, cams, Gs, walk=walk)
    ref = {f: np.zeros_like(g[f]) for f in PARAMS}
    for cam, G, img in zip(cams, Gs, imgs):
        assert np.abs(img - oracle.render_walk(sc, cam)).max() <= 1e-4
        gr, _ = oracle.adjoint_gradients(sc, cam, G)
        for f in PARAMS:
            ref[f] += gr[f].reshape(ref[f].shape)
    for f in PARAMS:
        assert_grad_close(g[f], ref[f], f)
