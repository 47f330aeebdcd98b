"""GPU: shooting by patches (power series shared by 32 x 32 rays) against
shooting ray by ray, which the entry point that allocates nothing and maps that
return the rays' positions use.

Ray-shooting counts must be equal: rays within 1e-6 pixels of a pixel's edge are
shot ray by ray in both.  IPM maps differ by the positions' rounding: the series
are cut below half a unit in the last place of the positions (at most ~100
theta_*, 1.4e-14, so below 1e-11 pixels here), and a pixel's deposits change by
less than ~4 times that relative to a cell's extent in pixels (at least 0.01
here), 4e-9 of a pixel that few cells feed; in the 2-norm over the map it
averages to well below 1e-9.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = {
    # name: (lens arguments, stars, request)
    "inside_the_disc": (dict(), 300, dict(hw1=1.0, hw2=1.0, n1=100, n2=90, rays_per_pixel=30.0)),
    "disc_edge": (dict(), 40, dict(y1c=7.6, y2c=2.1, hw1=3.0, hw2=2.0, n1=60, n2=60, nray1=1501, nray2=1307, x1c=9.0, x2c=6.0, dx1=4.0,
                                   dx2=4.0)),
    "beyond_the_disc": (dict(), 40, dict(y1c=25.5, y2c=1.0, hw1=3.0, hw2=2.0, n1=60, n2=60, nray1=1111, nray2=999, x1c=30.0, x2c=3.0,
                                         dx1=3.0, dx2=3.0)),
    "rectangle": (dict(sheet="rect", rect_aspect=1.7), 200, dict(hw1=1.0, hw2=1.0, n1=64, n2=64, nray1=2033,
                                                                 nray2=2500, dx1=6.0, dx2=9.0)),
    "rectangle_edge": (dict(sheet="rect", rect_aspect=0.8), 30, dict(hw1=4.0, hw2=2.5, n1=64, n2=64, nray1=1400,
                                                                     nray2=1200, dx1=9.0, dx2=7.0)),
    "no_sheet": (dict(sheet="none"), 100, dict(hw1=1.0, hw2=1.5, n1=50, n2=75, rays_per_pixel=200.0)),
    "one_star": (dict(), 1, dict(hw1=1.0, hw2=1.0, n1=40, n2=40, nray1=403, nray2=389, dx1=2.0, dx2=2.0)),
    "third_order": (dict(psi3=(0.001, 0.0, -0.002, 0.004)), 100, dict(hw1=1.0, hw2=1.0, n1=64, n2=64, nray1=1999,
                                                                      nray2=1801, x1c=0.5, x2c=0.2, dx1=4.0,
                                                                      dx2=4.0)),
    "unequal_spacing": (dict(), 100, dict(hw1=1.0, hw2=1.0, n1=64, n2=64, nray1=3001, nray2=601, dx1=4.0, dx2=4.0)),
    "low_order": (dict(), 200, dict(hw1=1.0, hw2=1.0, n1=64, n2=64, rays_per_pixel=60.0, order=5)),
    "top_order": (dict(), 200, dict(hw1=1.0, hw2=1.0, n1=64, n2=64, rays_per_pixel=60.0, order=31)),
}


def _lens(name):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    kw, n, req = CASES[name]
    if kw.get("sheet") == "rect":
        sf = W.rect_field(n, 0.3, kw["rect_aspect"], "salpeter", seed=11)
    else:
        sf = W.star_field(n, 0.3, "salpeter", seed=11)
    return mlm.Lens(0.3, 0.1, 0.25, sf.x, sf.y, sf.m, **kw), req


@pytest.mark.parametrize("name", list(CASES))
def test_irs_counts_equal_ray_by_ray(name):
    lens, req = _lens(name)
    got, st = lens.map(mapping="irs", **req)
    ref, sr = lens.map(mapping="irs", noalloc=True, **req)
    assert st["n_tiles"] < sr["n_tiles"] / 4   # by patches there, by tiles of 64 rays here
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
    assert st["n_tiles"] < sr["n_tiles"] / 4
    assert float((out - ref).norm() / ref.norm()) < 1e-9


def test_rows_add_up():
    lens, req = _lens("rectangle")
    whole, _ = lens.map(mapping="irs", **req)
    R = lens.region(**req)
    cut = R["nr2"] // 2 + 5
    a, _ = lens.map(mapping="irs", rows=(0, cut), **req)
    b, _ = lens.map(mapping="irs", rows=(cut, R["nr2"] - 1), **req)
    assert np.abs(a + b - whole).max() < 1e-12 * whole.max()
