"""The two composites of the rasteriser against one another where lists are long.

One view of few tiles goes to the sixteen-wave composite; thousands of copies of
it in one call, all with equal lists, go to the other.  That they do is asserted:
the sixteen-wave composite drops more cells before it tests them pixel by pixel,
so a copy's share of the tested (wave, cell) steps is larger.  Lists that fill the
ring of results many times, and lists of two culling steps (1024 entries each).
Equal bit for bit, images and record counts, as both do the same arithmetic in the
same order; and against the float64 oracle at 1e-4."""
import numpy as np
import pytest
import torch

import oracle
from column_scene import column_camera, column_scene

pytestmark = pytest.mark.gpu


# cells per tile, copies without and with records (at most 4096 cameras)
@pytest.mark.parametrize("length,copies,recorded", [(300, 1500, 1500), (700, 3800, 3800), (1150, 4000, 4000),
                                                    (1500, 6000, 0)])
def test_one_view_equals_many(length, copies, recorded):
    import paper_2604_24994_amd as pf
    print(f"case two tiles of lists of {length} or more, {copies} copies", flush=True)
    sc, depth = column_scene(2 * length, 4, seed=3)
    cam = column_camera(depth, 32, 8, 2)
    scene = pf.build_scene(sc, sigma_scale=sc.sigma_scale, tau=sc.tau)
    k = torch.zeros(6, dtype=torch.int64, device="cuda")
    one = pf.render_raster(scene, cam, counters=k)[0].clone()
    steps_one = int(k[3])
    k.zero_()
    many = pf.render_raster(scene, [cam] * copies, counters=k)
    steps_many = int(k[3]) / copies
    print(f"  steps of one view {steps_one}, of a copy {steps_many:.1f}")
    assert steps_many > steps_one and steps_many == int(steps_many)
    assert all(torch.equal(one, many[i]) for i in (0, 1, copies // 2, copies - 1))
    pix = np.array([3, 90, 160, 250])
    ref = oracle.render_walk(sc, cam, pix)
    assert np.abs(one.reshape(-1, 4)[pix].cpu().numpy() - ref).max() <= 1e-4
    if recorded:
        k.zero_()
        img, st = pf.render_raster_state(scene, cam)
        rec = st.info()["records"]
        st.release()
        imgs, st = pf.render_raster_state(scene, [cam] * recorded)
        assert torch.equal(img.view_as(one), one) and torch.equal(imgs.view(recorded, -1)[-1], img)
        assert st.info()["records"] == recorded * rec > 0
        st.release()
    scene.destroy()
