"""The ball that bounds a cell's dense part must never cut what the cell shows.

The ball is formed by the build from the faces' largest displacements, while
every render reads the texture as it is then.  Displacements far beyond the
cell, to either side, displacements raised in place after the build, and
normals without a direction, each against the float64 oracle or a fresh build.

Bars: 1e-4 per pixel against the oracle, as everywhere; 1e-6 against a fresh
build (the same pieces in the same order)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from conftest import assert_grad_close

pytestmark = pytest.mark.gpu

PARAMS = ("p", "power", "radius", "normal", "occ_logit", "rgb", "tex")


def _scene(n=240, seed=11):
    sc = W.scene_uniform(n, seed=seed)
    sc.radius = (sc.radius * 2.5).astype(np.float32)
    cam = W.pinhole(W.random_eyes(1, 2.7, seed)[0], 40, 33, 55.0)
    return sc, cam


def _box(cam):
    eye = np.asarray(cam.c2w)[:, 3]
    return np.minimum(eye, -1.6) - 0.1, np.maximum(eye, 1.6) + 0.1


def _images(pf, scene, cam):
    return {"raster": pf.render_raster(scene, cam)[0].cpu().numpy(),
            "walk": pf.render_trace(scene, cam)[0].cpu().numpy()}


def _grads(pf, scene, cam, state_of):
    img, st = state_of(scene, cam)
    g = torch.Generator().manual_seed(3)
    G = torch.randn(img.numel(), generator=g).to("cuda")
    d = {f: torch.zeros_like(scene.params[f]) for f in PARAMS}
    pf.backward(scene, st, G, d)
    st.release()
    return G.cpu().numpy().reshape(-1, 4).astype(np.float64), {f: t.cpu().numpy() for f, t in d.items()}


@pytest.mark.parametrize("disp", [0.3, -0.3, "mixed", "one site"])
def test_large_displacements_match_oracle(disp):
    import paper_2604_24994_amd as pf
    print(f"case displacements {disp}", flush=True)
    sc, cam = _scene()
    sc.tex = np.array(sc.tex)
    if disp == "mixed":
        sc.tex[:, :, 2] *= 5.0
    elif disp == "one site":
        sc.tex[:, :, 2] = -0.3
        sc.tex[:, 5, 2] = 0.3
    else:
        sc.tex[:, :, 2] += np.float32(disp)
    scene = pf.build_scene(sc, box=_box(cam))
    ref = oracle.render_painter(sc, cam).reshape(cam.height, cam.width, 4)
    assert ref[..., 3].max() > 0.1
    for name, img in _images(pf, scene, cam).items():
        print(f"  {name} {np.abs(img - ref).max():.2e}")
        assert np.abs(img - ref).max() <= 1e-4, name
    scene.destroy()


@pytest.mark.parametrize("n", [240, 20000])
def test_displacements_raised_in_place(n):
    import paper_2604_24994_amd as pf
    print(f"case {n} cells, displacements raised after the build", flush=True)
    sc, cam = _scene(n)
    sc.tex = np.array(sc.tex)
    sc.tex[:, :, 2] = -0.05          # most dense parts end below the face
    params = pf.to_device_params(sc)
    scene = pf.build_scene(params, sigma_scale=sc.sigma_scale, tau=sc.tau, box=_box(cam))
    low = _images(pf, scene, cam)
    up = torch.full((n, 8), 0.2, device="cuda")
    up[1::3] = -0.05                 # two cells of three
    up[0::3, 4] = 0.3
    scene.params["tex"][:, :, 2] = up
    sc.tex[:, :, 2] = up.cpu().numpy()
    fresh = pf.build_scene({f: t.clone() for f, t in scene.params.items()}, sigma_scale=sc.sigma_scale, tau=sc.tau,
                           box=_box(cam))
    ref = _images(pf, fresh, cam)
    both = _images(pf, scene, cam)
    for name in ref:
        assert np.abs(ref[name] - low[name]).max() > 1e-2
        print(f"  {name} {np.abs(both[name] - ref[name]).max():.2e}")
        assert np.abs(both[name] - ref[name]).max() <= 1e-6, name
    if n == 240:
        for f in (pf.render_raster_state, pf.render_trace_state):
            G, g = _grads(pf, scene, cam, f)
            gr, _ = oracle.adjoint_gradients(sc, cam, G)
            for a in PARAMS:
                assert_grad_close(g[a], gr[a], a)
    # back again: the first image
    scene.params["tex"][:, :, 2] = -0.05
    for name, img in _images(pf, scene, cam).items():
        assert np.abs(img - low[name]).max() <= 1e-6, name
    scene.destroy()
    fresh.destroy()


def test_displacements_raised_in_place_walk_alone():
    # the walk alone, and its form without allocations
    import paper_2604_24994_amd as pf
    print("case displacements raised after the build, walks only", flush=True)
    sc, cam = _scene(600, 5)
    sc.tex = np.array(sc.tex)
    sc.tex[:, :, 2] = -0.05
    for noalloc in (False, True):
        scene = pf.build_scene(sc, box=_box(cam))
        scene.params["tex"][:, :, 2] = 0.2
        fresh = pf.build_scene({f: t.clone() for f, t in scene.params.items()}, sigma_scale=sc.sigma_scale,
                               tau=sc.tau, box=_box(cam))
        want = pf.render_trace(fresh, cam)[0]
        if noalloc:
            out = torch.empty(cam.n_rays * 4, device="cuda")
            got = pf.render_trace_noalloc(scene, cam, out)[0]
        else:
            got = pf.render_trace(scene, cam)[0]
        assert float((got.reshape(-1) - want.reshape(-1)).abs().max()) <= 1e-6, noalloc
        scene.destroy()
        fresh.destroy()

@pytest.mark.parametrize("kind", ["zero", "nan", "inf", "tiny"])
def test_normal_without_direction_leaves_the_cell_dense(kind):
    # Without a direction no face cuts the cell: all of it is dense, and its
    # sites weigh alike (given one texture here, so that no weights matter).
    # The reference has a face moved out of the cell instead.
    import paper_2604_24994_amd as pf
    print(f"case normal {kind}", flush=True)
    sc, cam = _scene()
    sc.tex = np.array(sc.tex)
    sc.tex[:, :, 3:] = sc.tex[:, :1, 3:]
    cells = np.arange(0, sc.n, 7)
    ref_sc = sc.copy()
    ref_sc.tex = np.array(ref_sc.tex)
    ref_sc.tex[cells, :, 2] = 10.0
    ref = oracle.render_painter(ref_sc, cam).reshape(cam.height, cam.width, 4)
    assert np.abs(oracle.render_painter(sc, cam).reshape(ref.shape) - ref).max() > 1e-2
    sc.normal = np.array(sc.normal)
    sc.normal[cells] = {"zero": 0.0, "nan": np.nan, "inf": np.inf, "tiny": 0.0}[kind]
    if kind == "tiny":
        sc.normal[cells, 1] = 1e-30   # its length is 0 in float32
    scene = pf.build_scene(sc, box=_box(cam))
    for name, img in _images(pf, scene, cam).items():
        print(f"  {name} {np.abs(img - ref).max():.2e}")
        assert np.abs(img - ref).max() <= 1e-4, name
    scene.destroy()
