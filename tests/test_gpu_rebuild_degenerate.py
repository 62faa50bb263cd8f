"""Rebuilds of sites moved into degenerate positions give the fresh build's scene.

Sites flattened into a plane or onto a lattice: the normals of a cell's old
planes become coplanar, so that nothing but rounding is left of what proved an
empty cell empty, and vertices, distances and offsets tie.  The adjacency must
come out equal to a fresh build's, which looks at every site."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

MOVES = {
    "plane z = x": lambda p: torch.stack([p[:, 0], p[:, 1], p[:, 0]], 1),
    "plane z = 2 x": lambda p: torch.stack([p[:, 0], p[:, 1], 2.0 * p[:, 0]], 1),
    "plane z = x + y": lambda p: torch.stack([p[:, 0], p[:, 1], p[:, 0] + p[:, 1]], 1),
    "plane z = 0": lambda p: torch.stack([p[:, 0], p[:, 1], 0.0 * p[:, 0]], 1),
    "nearly flat": lambda p: torch.stack([p[:, 0], p[:, 1], p[:, 2] / 4096.0], 1),
    "lattice of 1/8": lambda p: torch.round(p * 8.0) / 8.0,
    "lattice of 1/64": lambda p: torch.round(p * 64.0) / 64.0,
}


@pytest.mark.parametrize("name", list(MOVES))
@pytest.mark.parametrize("seed", [4, 5])
def test_rebuild_equals_fresh_build(name, seed):
    import paper_2604_24994_amd as pf
    print(f"case 30,000 cells to {name}, seed {seed}", flush=True)
    params = pf.to_device_params(W.scene_mixture(30000, seed=seed))
    scene = pf.build_scene(params)
    moved = dict(params)
    moved["p"] = MOVES[name](params["p"]).contiguous()
    for _ in range(2):   # (the second rebuild starts from the degenerate scene)
        pf.update_scene(scene, moved)
        fresh = pf.build_scene(moved)
        (r0, c0), (r1, c1) = scene.adjacency(), fresh.adjacency()
        assert torch.equal(r0, r1) and torch.equal(c0, c1)
        assert scene.info()["n_hidden"] == fresh.info()["n_hidden"]
        fresh.destroy()
    scene.destroy()


@pytest.mark.parametrize("n", [23999, 24000, 24001])
def test_sizes_where_empty_cells_start_to_be_taken_out(n):
    import paper_2604_24994_amd as pf
    print(f"case {n} cells, sites moved by 1e-3", flush=True)
    params = pf.to_device_params(W.scene_uniform(n, seed=4))
    scene = pf.build_scene(params)
    g = torch.Generator(device="cuda").manual_seed(n)
    for _ in range(2):
        params = dict(params, p=params["p"] + 1e-3 * torch.randn(n, 3, device="cuda", generator=g))
        pf.update_scene(scene, params)
        fresh = pf.build_scene(params)
        (r0, c0), (r1, c1) = scene.adjacency(), fresh.adjacency()
        assert torch.equal(r0, r1) and torch.equal(c0, c1)
        fresh.destroy()
    scene.destroy()
