"""The two composites of the rasteriser give the same pixels.

A single small view is composited by sixteen waves per 8x8 quadrant (its
tiles cannot fill the chip); the same view repeated many times in one call is
composited by one wave per quadrant (no list is longer than the launch's
share).  Both run the same arithmetic in the same order per pixel, so the
images are equal bit for bit, and so are the record counts."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

CASES = {
    # lists of a few entries, image edges inside a tile and inside a quadrant
    "1k cells 100x67": (lambda: W.scene_uniform(1024), lambda e: W.pinhole(e, 100, 67, 60.0), 3.0),
    # many cells per pixel: lists of several culling steps, the result ring used many times over
    "40k cells 40x24": (lambda: W.scene_mixture(40000, seed=3), lambda e: W.pinhole(e, 40, 24, 60.0), 4.0),
    "40k cells fisheye 33x49": (lambda: W.scene_mixture(40000, seed=3), lambda e: W.fisheye(e, 33, 49, 180.0), 4.0),
    # a camera inside the scene: balls around and behind it
    "4k cells from inside": (lambda: W.scene_uniform(4096, seed=5), lambda e: W.pinhole(e, 64, 64, 90.0), 0.2),
    # a quadrant wider than the cone test takes
    "1k cells fisheye 8x8": (lambda: W.scene_uniform(1024), lambda e: W.fisheye(e, 8, 8, 180.0), 1.0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_one_view_equals_many(name):
    import paper_2604_24994_amd as pf
    print(f"case {name}: one view against 512 copies of it in one call", flush=True)
    make, cam_of, dist = CASES[name]
    sc = make()
    cam = cam_of(W.random_eyes(1, dist, 2)[0])
    scene = pf.build_scene(sc)
    one = pf.render_raster(scene, cam)[0]
    many = pf.render_raster(scene, [cam] * 512)
    assert float(one[..., 3].max()) > 0.0
    for i in (0, 1, 255, 511):
        assert torch.equal(one, many[i]), (name, i)
    img, st = pf.render_raster_state(scene, cam)
    imgs, st4 = pf.render_raster_state(scene, [cam] * 512)
    assert torch.equal(img.view_as(one), one) and torch.equal(imgs[:img.numel()], img)
    assert st4.info()["records"] == 512 * st.info()["records"] > 0
    st.release()
    st4.release()
    scene.destroy()
