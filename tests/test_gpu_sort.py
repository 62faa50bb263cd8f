"""Tile lists around the lengths at which their sort changes: in the LDS of a
small workgroup, in that of a large one, and run by run.  All cells fall into one
16x16 tile, so the list is as long as the scene; compositing in another order
than by depth would show, so the image is held to the walk's (no lists) at
1e-4, the library's bar against its float64 oracle."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096, 4097, 16384, 16385, 33000])
def test_one_tile_sorted(n):
    import paper_2604_24994_amd as pf
    print(f"case one tile of {n} cells", flush=True)
    sc = W.scene_uniform(n, seed=9)
    cam = W.pinhole(np.array([0.3, -0.2, 5.0]), 16, 16, 45.0)
    scene = pf.build_scene(sc, box=((-6.0,) * 3, (6.0,) * 3))
    ras = pf.render_raster(scene, cam)[0].cpu().numpy()
    trc = pf.render_trace(scene, cam)[0].cpu().numpy()
    assert ras[..., 3].max() > 0.0
    print(f"  raster-walk {np.abs(ras - trc).max():.2e}")
    assert np.abs(ras - trc).max() <= 1e-4
    scene.destroy()
