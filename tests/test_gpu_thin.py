"""GPU: cells with a triangle thinner than 2^-16 pixels, whose vertices are shot
ray by ray although the grid is shot by patches.

A triangle's deposits are quotients by its area, so an error d of its vertices'
positions changes them by d / thickness.  The positions of both ways differ by
rounding: 8 units in the last place (1.8e-15 each) of positions up to 16 theta_*,
2.9e-14 theta_*, 4.3e-13 pixels of 1/15 theta_*.  A triangle of 2^-16 pixels then
changes by 4.3e-13 * 65536 = 2.8e-8 of its weight, and few such triangles meet in
a pixel: 1e-7 of a triangle's weight bounds every pixel.  Triangles that stretch
over many pixels are the ones whose deposits cancel; the field of the second test
holds one.
"""
import math

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [1, 2, 3])
@pytest.mark.parametrize("n", [300, 240])   # 22 cells a pixel and 34: the cell pass's two windows
def test_thin_cells_equal_ray_by_ray(seed, n):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    sf = W.star_field(60, 0.3, "salpeter", seed=seed)
    lens = mlm.Lens(0.3, 0.1, 0.25, sf.x, sf.y, sf.m, sheet="none")
    req = dict(hw1=10.0 * n / 300, hw2=10.0 * n / 300, n1=n, n2=n, nray1=1501, nray2=1307, dx1=8.0, dx2=8.0)
    R = lens.region(**req)
    out = torch.empty((n, n), dtype=torch.float64, device="cuda")
    ref = torch.empty_like(out)
    w = torch.empty((R["nr2"], R["nr1"], 2), dtype=torch.float64, device="cuda")
    _, st = lens.map(out=out, **req)
    _, sr = lens.map(out=ref, w_out=w, **req)
    assert st["n_tiles"] < sr["n_tiles"] / 2   # by patches there, by tiles of 64 rays here
    # pixel coordinates of the rays: some cells are thin, and lie in the map
    p = (w + 10.0 * n / 300) * 15.0
    d, e, f = p[1:, 1:] - p[:-1, :-1], p[:-1, 1:] - p[:-1, :-1], p[1:, :-1] - p[:-1, :-1]
    s1, s2 = e[..., 0] * d[..., 1] - d[..., 0] * e[..., 1], d[..., 0] * f[..., 1] - f[..., 0] * d[..., 1]
    thin = torch.minimum(s1 * s1, s2 * s2) < (d * d + e * e + f * f).sum(-1) / 65536.0 ** 2
    inside = ((p > 0) & (p < n)).all(-1)[:-1, :-1]
    assert int((thin & inside).sum()) > 50
    weight = 0.5 * (16.0 / 1500) * (16.0 / 1306) * 15.0 ** 2
    assert float((out - ref).abs().max()) < 1e-7 * weight


def test_long_thin_triangle():
    """The paper's Table 1 map, a rectangle of stars; positions up to 64
    theta_* (units of 1.4e-14) and pixels of 0.01: 8 half units are 5.7e-12 pixels,
    3.7e-7 of a triangle's weight at 2^-16 pixels, and four of them in a pixel."""
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    r = math.sqrt(0.6 / 1e-3)
    a, b = 10.0 + r, (10.0 + r) / 0.2
    field = mlm.field_params(0.6, "equal", n_stars=int(round(0.6 * 4 * 1.2 * a * 1.2 * b / math.pi)), seed=103947,
                             shape="rect", rect_aspect=b / a)
    lens = mlm.Lens.sampled(0.6, 0.0, 0.6, field, sheet="rect")
    req = dict(hw1=10.0, hw2=10.0, n1=2000, n2=2000, flux_fraction=1e-3)
    R = lens.region(**req)
    out = torch.empty((2000, 2000), dtype=torch.float64, device="cuda")
    ref = torch.empty_like(out)
    w = torch.empty((R["nr2"], R["nr1"], 2), dtype=torch.float64, device="cuda")
    _, st = lens.map(out=out, **req)
    _, sr = lens.map(out=ref, w_out=w, **req)
    assert st["n_tiles"] < sr["n_tiles"] / 2
    weight = 0.5 * R["d1"] * R["d2"] / (R["pix1"] * R["pix2"])
    assert float((out - ref).abs().max()) < 4 * 3.7e-7 * weight
