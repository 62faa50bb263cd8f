"""The walk's deferred radiance: a wave evaluates pending contributions cell by
cell on the matrix cores, or ray by ray where few rays share a cell, whenever
a ray's ring of ten is full and once more at the end.

Bar: image against the rasteriser's within 1e-4, the library's bar against its
float64 oracle.  The record-writing walk runs the same arithmetic in the same
order, so its image is equal bit for bit, and the gradients agree with the
rasteriser's to 1e-5 in norm, as for any two orders of the same sums."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

PARAMS = ("p", "power", "radius", "normal", "occ_logit", "rgb", "tex")

CASES = {
    # every ray of a wave in the same few cells; image edges inside a wave
    "64 cells narrow 41x27": (lambda: W.scene_uniform(64), lambda e: W.pinhole(e, 41, 27, 12.0), 3.0),
    # many contributions per ray (the ring is used many times over), neighbours apart
    "20k cells 24x40": (lambda: W.scene_mixture(20000, seed=3), lambda e: W.pinhole(e, 24, 40, 60.0), 4.0),
    # hardly two rays in one cell: the ray-by-ray branch
    "20k cells fisheye 16x16": (lambda: W.scene_mixture(20000, seed=3), lambda e: W.fisheye(e, 16, 16, 180.0), 0.4),
    # one pixel: one ray of the wave walks
    "1k cells 1x1": (lambda: W.scene_uniform(1024), lambda e: W.pinhole(e, 1, 1, 5.0), 3.0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_walk_equals_raster_and_its_record_form(name):
    import paper_2604_24994_amd as pf
    print(f"case {name}", flush=True)
    make, cam_of, dist = CASES[name]
    sc = make()
    cam = cam_of(W.random_eyes(1, dist, 2)[0])
    scene = pf.build_scene(sc, box=((-6.0,) * 3, (6.0,) * 3))
    ras = pf.render_raster(scene, cam)[0].cpu().numpy()
    k = torch.zeros(6, dtype=torch.int64, device="cuda")
    trc = pf.render_trace(scene, cam, counters=k)[0].cpu().numpy()
    assert ras[..., 3].max() > 0.0
    print(f"  contributions per ray {int(k[3]) / max(1, int(k[0])):.1f}, raster-walk {np.abs(ras - trc).max():.2e}")
    assert np.abs(ras - trc).max() <= 1e-4
    g = torch.Generator().manual_seed(5)
    G = torch.randn(cam.height * cam.width * 4, generator=g).to("cuda")
    grads = []
    for f in (pf.render_trace_state, pf.render_raster_state):
        img, st = f(scene, cam)
        if not grads:
            assert np.array_equal(img.cpu().numpy().reshape(trc.shape), trc)
        d = {a: torch.zeros_like(scene.params[a]) for a in PARAMS}
        pf.backward(scene, st, G, d)
        grads.append({a: b.double().cpu() for a, b in d.items()})
        st.release()
    for a in PARAMS:
        x, y = grads[0][a], grads[1][a]
        r = float((x - y).norm() / y.norm().clamp_min(1e-300))
        print(f"  {a}: rel {r:.2e}")
        assert r <= 1e-5, a
    # cut short: as many steps, whatever is pending is still added
    for n in (1, 7):
        a, cut = pf.render_trace(scene, cam, max_steps=n, return_truncated=True)
        b, st = pf.render_trace_state(scene, cam, max_steps=n)
        assert torch.equal(a[0].reshape(-1), b.reshape(-1))
        st.release()
    scene.destroy()
