"""The backward of cells with many faces: planes and sums in LDS (up to 64 faces),
sums alone (up to 128), the rest in global memory.  One large cell amid small ones
that are all its neighbours, against the float64 oracle adjoint at the
repository's gradient bar."""
import numpy as np
import pytest

import oracle
import workloads as W
from conftest import assert_grad_close
from test_gpu_modes import PARAMS, _grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("faces", [64, 65, 128, 129, 180])
def test_large_cell_matches_oracle(faces):
    import paper_2604_24994_amd as pf
    print(f"case one cell of {faces} faces", flush=True)
    sc = W.scene_uniform(faces + 1, seed=6)
    # neighbours spread evenly over a sphere: each has a face within it
    k = np.arange(faces)
    z = 1.0 - (2.0 * k + 1.0) / faces
    t = np.pi * (1.0 + 5.0 ** 0.5) * k
    d = np.stack([np.sqrt(1.0 - z * z) * np.cos(t), np.sqrt(1.0 - z * z) * np.sin(t), z], 1)
    sc.p[0] = 0.0
    sc.p[1:] = (0.8 * d + 0.003 * np.random.default_rng(2).normal(size=d.shape)).astype(np.float32)
    sc.radius[:] = 0.1
    sc.radius[0] = 1.5
    sc.power[:] = 0.0
    scene = pf.build_scene(sc)
    row, col = scene.adjacency()
    assert int(row[1] - row[0]) == faces and int((col[:faces] >= 0).sum()) == faces
    scene.destroy()
    cam = W.pinhole(W.random_eyes(1, 2.7, 3)[0], 26, 22, 40.0)
    G = np.random.default_rng(7).normal(size=(cam.n_rays, 4))
    g, _ = _grads(pf, sc, [cam], [G])
    ref, _ = oracle.adjoint_gradients(sc, cam, G)
    for f in PARAMS:
        assert np.abs(ref[f]).max() > 0.0
        assert_grad_close(g[f], ref[f], f)
