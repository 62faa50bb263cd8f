"""Rebuilding a scene in place gives the scene a fresh build gives.

The rebuild first takes out the cells that the previous build found empty and
whose four witness planes still leave nothing of them; everything else is
clipped without those sites.  The adjacency must come out equal to a fresh
build's (which looks at every site), for small moves (nearly all witnesses
hold), large ones (many fail), none, several in a row, sizes around the
limit below which no cell is taken out, and changed weights."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _same(pf, scene, params, sc):
    fresh = pf.build_scene(params, sigma_scale=sc.sigma_scale, tau=sc.tau)
    r0, c0 = scene.adjacency()
    r1, c1 = fresh.adjacency()
    assert torch.equal(r0, r1) and torch.equal(c0, c1)
    i0, i1 = scene.info(), fresh.info()
    assert i0["n_hidden"] == i1["n_hidden"] and i0["n_faces"] == i1["n_faces"]
    cam = W.pinhole(W.random_eyes(1, 4.0, 1)[0], 96, 64, 60.0)
    a, b = pf.render_raster(scene, cam)[0], pf.render_raster(fresh, cam)[0]
    # the same faces; a cell's bounds may differ in the last bit (vertices from other triples of planes)
    assert float((a - b).abs().max()) <= 1e-6
    fresh.destroy()
    return int(i0["n_hidden"])


@pytest.mark.parametrize("n,move", [(16383, 1e-3), (16384, 1e-4), (16385, 1e-2), (50000, 0.0), (50000, 0.1)])
def test_rebuild_equals_fresh_build(n, move):
    import paper_2604_24994_amd as pf
    print(f"case rebuild: {n} cells, sites moved by {move} three times", flush=True)
    sc = W.scene_mixture(n, seed=4)
    rng = np.random.default_rng(4)
    params = pf.to_device_params(sc)
    scene = pf.build_scene(params, sigma_scale=sc.sigma_scale, tau=sc.tau)
    for _ in range(3):
        params = dict(params)
        step = torch.tensor(rng.normal(scale=move, size=sc.p.shape).astype(np.float32), device="cuda")
        params["p"] = params["p"] + step
        pf.update_scene(scene, params)
        assert _same(pf, scene, params, sc) > 0
    # other weights and radii: cells empty before are empty no more, and the other way round
    params = dict(params)
    s = torch.tensor(rng.uniform(0.02, 0.1, size=n).astype(np.float32), device="cuda")
    params["power"], params["radius"] = s * s, 1.5 * s
    pf.update_scene(scene, params)
    _same(pf, scene, params, sc)
    # two sites at one place, one of them heavier
    params = dict(params)
    p = params["p"].clone()
    p[1::2] = p[0::2][:p[1::2].shape[0]]
    params["p"] = p
    pf.update_scene(scene, params)
    _same(pf, scene, params, sc)
    pf.update_scene(scene, params)
    _same(pf, scene, params, sc)
    scene.destroy()
