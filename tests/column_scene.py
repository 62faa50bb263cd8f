"""Scenes whose tile lists have a wanted length (shared by the tests of the lists
and of the two composites)."""
import numpy as np

import workloads as W

PITCH, STEP = 0.5, 0.02


def column_scene(n, side, seed=0):
    """n cells in side x side columns along z, thin slabs stacked with faces
    nearly across z, so that every ray of a view along z meets every cell of its
    column, each a little opaque."""
    rng = np.random.default_rng(seed)
    sc = W.scene_uniform(n, seed=seed)
    k = np.arange(n)
    col, lev = k % (side * side), k // (side * side)
    depth = STEP * (lev.max() + 1)
    p = np.stack([PITCH * (col % side - (side - 1) / 2), PITCH * (col // side - (side - 1) / 2),
                  STEP * (lev + 0.6 * rng.uniform(size=side * side)[col])], 1)
    sc.p = np.ascontiguousarray(p[rng.permutation(n)], dtype=np.float32)
    sc.power[:], sc.radius[:] = 0.0, 0.45
    sc.normal[:] = 0.05 * rng.normal(size=(n, 3))
    sc.normal[:, 2] = np.where(rng.uniform(size=n) < 0.5, -1.0, 1.0)
    sc.tex = np.array(sc.tex)
    sc.tex[:, :, 2] *= 0.02
    sc.occ_logit[:] = rng.uniform(-1.0, 1.0, size=n)
    sc.sigma_scale = float(4.0 / (0.7 * depth))
    return sc, depth


def column_camera(depth, width, height, across):
    """A view along z from afar: 16 pixels see ``across`` columns."""
    dist = 40.0 + 10.0 * depth
    cam = W.pinhole(np.array([0.0, 0.0, -dist]), width, height, 10.0)
    cam.c2w = np.concatenate([np.eye(3), [[0.0], [0.0], [-dist]]], 1).astype(np.float32)
    cam.fx = cam.fy = 16.0 / (PITCH * across) * (dist + 0.5 * depth)
    return cam
