"""GPU: shooting by patches where leaves are smaller than a patch, against shooting
ray by ray (the entry point that allocates nothing, and maps that return the rays'
positions).

A tight group of stars has leaves of every size around it, down to less than a
ray's distance, while the mean number of rays per leaf is that of the sparse
stars, so the grid is shot by patches.  Bounds as in test_gpu_patch.py: equal
counts; IPM maps within 1e-9 in the 2-norm (positions of at most 16 theta_*,
1.8e-15 a unit in the last place, over cells at least 0.01 pixels wide).
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = {
    # name: (sparse stars, stars of the group, its radius, request)
    "group_16": (12, 40, 1e-3, dict(n1=60, n2=50, nray1=1701, nray2=1603)),
    "group_32": (12, 40, 1e-3, dict(n1=60, n2=50, nray1=2801, nray2=2707)),
    "group_64": (12, 40, 1e-3, dict(n1=60, n2=50, nray1=8001, nray2=7907)),
    "pair_16": (3, 2, 4e-3, dict(n1=60, n2=50, nray1=1901, nray2=1803, leaf_max=1)),
    "pair_32": (3, 2, 4e-3, dict(n1=60, n2=50, nray1=2801, nray2=2707, leaf_max=1)),
    "coincident": (12, 40, 0.0, dict(n1=60, n2=50, nray1=2401, nray2=2307, max_level=12)),
}


def _lens(name):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    n, group, radius, req = CASES[name]
    sf = W.star_field(n, 0.3, "salpeter", seed=7)
    r = np.random.default_rng(8)
    e = radius * r.uniform(-1, 1, (2, group))
    x, y = np.concatenate([sf.x, 0.613 + e[0]]), np.concatenate([sf.y, -0.337 + e[1]])
    m = np.concatenate([sf.m, np.full(group, 1e-3 / group)])   # (light: the rays beside it land in the map)
    # (a stated order: beyond 24 the many terms exclude the patch by themselves)
    req = dict(dict(hw1=1.5, hw2=1.25, dx1=3.0, dx2=3.0, order=20), **req)
    return mlm.Lens(0.3, 0.1, 0.25, x, y, m, sheet="none"), req


@pytest.mark.parametrize("name", list(CASES))
def test_irs_counts_equal_ray_by_ray(name):
    lens, req = _lens(name)
    got, st = lens.map(mapping="irs", **req)
    ref, sr = lens.map(mapping="irs", noalloc=True, **req)
    assert st["n_tiles"] < sr["n_tiles"] / 2   # by patches there, by tiles of 64 rays here
    assert np.array_equal(got, ref)
    assert ref.sum() > 0


@pytest.mark.parametrize("name", list(CASES))
def test_ipm_map_equals_ray_by_ray(name):
    import torch
    lens, req = _lens(name)
    R = lens.region(**req)
    out = torch.empty((req["n2"], req["n1"]), dtype=torch.float64, device="cuda")
    ref = torch.empty_like(out)
    w = torch.empty((R["nr2"], R["nr1"], 2), dtype=torch.float64, device="cuda")
    _, st = lens.map(out=out, **req)
    _, sr = lens.map(out=ref, w_out=w, **req)
    assert st["n_tiles"] < sr["n_tiles"] / 2
    assert float((out - ref).norm() / ref.norm()) < 1e-9


@pytest.mark.parametrize("mapping", ["ipm", "irs"])
@pytest.mark.parametrize("leaf_max,patches", [(32, True), (64, True), (256, False), (1000, False)])
def test_leaves_of_many_stars_are_shot_ray_by_ray(leaf_max, patches, mapping):
    """A patch takes at most 64 near stars of its leaf: where leaves mostly hold
    more, patches would be the slower way."""
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    sf = W.star_field(5000, 0.4, "salpeter", seed=3)
    lens = mlm.Lens(0.4, 0.1, 0.2, sf.x, sf.y, sf.m, sheet="none")
    req = dict(hw1=6.0, hw2=6.0, n1=100, n2=100, rays_per_pixel=400.0, leaf_max=leaf_max, mapping=mapping)
    got, st = lens.map(**req)
    ref, sr = lens.map(noalloc=True, **req)
    assert (st["n_tiles"] < sr["n_tiles"] / 2) == patches
    if mapping == "irs":
        assert np.array_equal(got, ref)
    else:
        assert np.linalg.norm(got - ref) < 1e-9 * np.linalg.norm(ref)
