"""The backward's branches: cameras and face planes held in LDS or read from
global memory, Spherical-Voronoi sums out of float32's range, a few records and
many (several batches and chunks of one cell).  Each against the float64 oracle
adjoint at the repository's gradient bar."""
import numpy as np
import pytest

import oracle
import workloads as W
from conftest import assert_grad_close
from test_gpu_modes import PARAMS, _grads

pytestmark = pytest.mark.gpu


def _many_cameras(k):
    sc = W.scene_uniform(60, seed=4)
    sc.radius = (sc.radius * 2.0).astype(np.float32)
    return sc, [W.pinhole(e, 9 + i, 7, 55.0) for i, e in enumerate(W.random_eyes(k, 2.7, 8))]


def _many_faces():
    # one large cell amid 120 small ones, all of them its neighbours
    sc = W.scene_uniform(121, seed=6)
    d = np.random.default_rng(2).normal(size=(120, 3))
    sc.p[0] = 0.0
    sc.p[1:] = (0.8 * d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    sc.radius[:] = 0.25
    sc.radius[0] = 1.5
    sc.power[:] = (sc.power * 0.0).astype(np.float32)
    return sc, [W.pinhole(e, 24, 18, 50.0) for e in W.random_eyes(1, 2.7, 3)]


def _large_axes():
    # logits of some hundreds: the unshifted sums overflow
    sc, cams = _many_cameras(2)
    sc.tex = np.array(sc.tex)
    m = (sc.tex.shape[2] - 3) // 6
    sc.tex[:, :, 3:3 + 3 * m] *= 60.0
    return sc, cams


def _one_cell():
    # more records than a workgroup takes, all of one cell
    sc = W.scene_uniform(2, seed=1)
    sc.radius[:] = 0.9
    return sc, [W.pinhole(e, 72, 64, 30.0) for e in W.random_eyes(1, 2.7, 5)]


CASES = {"8 cameras": lambda: _many_cameras(8), "9 cameras": lambda: _many_cameras(9), "120 faces": _many_faces,
         "large axes": _large_axes, "one cell": _one_cell}


@pytest.mark.parametrize("name", list(CASES))
def test_backward_branch_matches_oracle(name):
    import paper_2604_24994_amd as pf
    print(f"case {name}", flush=True)
    sc, cams = CASES[name]()
    rng = np.random.default_rng(7)
    Gs = [rng.normal(size=(c.n_rays, 4)) for c in cams]
    g, _ = _grads(pf, sc, cams, Gs)
    ref = {f: np.zeros_like(g[f]) for f in PARAMS}
    for cam, G in zip(cams, Gs):
        gr, _ = oracle.adjoint_gradients(sc, cam, G)
        for f in PARAMS:
            ref[f] += gr[f].reshape(ref[f].shape)
    for f in PARAMS:
        assert_grad_close(g[f], ref[f], f)
