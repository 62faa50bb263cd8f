"""Tile lists of known lengths around those at which their sort changes: in the
LDS of a small workgroup (up to 4096 entries), in that of a large one (16384), and
run by run with stages in global memory between, the last run of one entry or
more.

One tile sees columns of thin cells.  Every cell contributes to some pixel (its
contribution sum is asserted), so the tile's list holds all of them.  Bars: 1e-4
per pixel against the walk, which has no lists, and the float64 oracle; an entry
out of place weighs 1e-3."""
import numpy as np
import pytest
import torch

import oracle
from column_scene import column_camera, column_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096, 4097, 16384, 16385, 32768, 32769, 45000])
def test_list_of_n_entries(n):
    import paper_2604_24994_amd as pf
    print(f"case a list of {n} entries", flush=True)
    sc, depth = column_scene(n, 4)
    cam = column_camera(depth, 16, 16, 4)
    z = float(cam.c2w[2, 3])
    scene = pf.build_scene(sc, sigma_scale=sc.sigma_scale, tau=sc.tau, box=((-3.0, -3.0, z - 1.0), (3.0, 3.0, depth + 3.0)))
    ras = pf.render_raster(scene, cam)[0].cpu().numpy()
    trc = pf.render_trace(scene, cam)[0].cpu().numpy()
    img, st = pf.render_raster_state(scene, cam)
    seen = torch.zeros(n, device="cuda")
    grads = {f: torch.zeros_like(t) for f, t in scene.params.items()}
    pf.backward(scene, st, torch.ones_like(img), grads, contribution=seen)
    st.release()
    assert int((seen > 0).sum()) == n
    assert np.array_equal(img.cpu().numpy().reshape(ras.shape), ras)
    pix = np.array([0, 70, 185, 255])
    ref = oracle.render_walk(sc, cam, pix)
    print(f"  raster-walk {np.abs(ras - trc).max():.2e} oracle {np.abs(ras.reshape(-1, 4)[pix] - ref).max():.2e}")
    assert ras[..., 3].max() < 0.9999   # no ray ends early
    assert np.abs(ras - trc).max() <= 1e-4
    assert np.abs(ras.reshape(-1, 4)[pix] - ref).max() <= 1e-4
    scene.destroy()
