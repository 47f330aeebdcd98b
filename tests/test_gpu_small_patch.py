"""GPU: patches of 16 x 16 rays, where a leaf holds fewer rays than 32 x 32 patches
need, against shooting ray by ray; tolerances as for the larger patches."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = {
    "disc": (dict(), 600, dict(hw1=1.0, hw2=1.0, n1=100, n2=90, nray1=1201, nray2=1107, dx1=6.0, dx2=6.0)),
    "disc_edge": (dict(), 360, dict(y1c=7.6, y2c=2.1, hw1=3.0, hw2=2.0, n1=60, n2=60, nray1=801, nray2=707, x1c=13.0,
                                    x2c=6.0, dx1=5.0, dx2=4.0)),
    "rectangle": (dict(sheet="rect", rect_aspect=1.7), 500, dict(hw1=1.0, hw2=1.0, n1=64, n2=64, nray1=897, nray2=1001,
                                                                 dx1=5.0, dx2=5.0)),
    "no_sheet": (dict(sheet="none"), 500, dict(hw1=1.0, hw2=1.5, n1=50, n2=75, nray1=1000, nray2=1015, dx1=6.0, dx2=6.0)),
}


def _lens(name):
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    kw, n, req = CASES[name]
    if kw.get("sheet") == "rect":
        sf = W.rect_field(n, 0.3, kw["rect_aspect"], "salpeter", seed=11)
    else:
        sf = W.star_field(n, 0.3, "salpeter", seed=11)
    return mlm.Lens(0.3, 0.1, 0.25, sf.x, sf.y, sf.m, **kw), req


@pytest.mark.parametrize("name", list(CASES))
def test_equals_ray_by_ray(name):
    import torch
    lens, req = _lens(name)
    got, st = lens.map(mapping="irs", **req)
    ref, sr = lens.map(mapping="irs", noalloc=True, **req)
    # by patches of 256 rays here, by tiles of 64 there
    assert sr["n_tiles"] / 4.2 < st["n_tiles"] < sr["n_tiles"] / 3
    assert np.array_equal(got, ref) and ref.sum() > 0
    R = lens.region(**req)
    out = torch.empty((req["n2"], req["n1"]), dtype=torch.float64, device="cuda")
    exact = torch.empty_like(out)
    w = torch.empty((R["nr2"], R["nr1"], 2), dtype=torch.float64, device="cuda")
    lens.map(out=out, **req)
    lens.map(out=exact, w_out=w, **req)
    assert float((out - exact).norm() / exact.norm()) < 1e-9


LARGE = {
    "disc": (dict(), 60, dict(hw1=1.0, hw2=1.0, n1=100, n2=90, nray1=6001, nray2=5503, dx1=4.0, dx2=4.0)),
    "rectangle": (dict(sheet="rect", rect_aspect=1.7), 80, dict(hw1=1.0, hw2=1.0, n1=64, n2=64, nray1=5733, nray2=6000,
                                                                dx1=3.0, dx2=3.0)),
    "no_sheet": (dict(sheet="none"), 1, dict(hw1=1.0, hw2=1.5, n1=50, n2=75, nray1=5800, nray2=5815, dx1=3.0, dx2=3.0)),
}


@pytest.mark.parametrize("name", list(LARGE))
def test_large_patches_equal_ray_by_ray(name):
    """Patches of 64 x 64 rays, from some 260,000 rays a leaf on."""
    import torch
    CASES["large_" + name] = LARGE[name]
    lens, req = _lens("large_" + name)
    got, st = lens.map(mapping="irs", **req)
    ref, sr = lens.map(mapping="irs", noalloc=True, **req)
    assert sr["n_tiles"] / 66 < st["n_tiles"] < sr["n_tiles"] / 50      # 4096 rays against 64
    assert np.array_equal(got, ref) and ref.sum() > 0
    R = lens.region(**req)
    out = torch.empty((req["n2"], req["n1"]), dtype=torch.float64, device="cuda")
    exact = torch.empty_like(out)
    w = torch.empty((R["nr2"], R["nr1"], 2), dtype=torch.float64, device="cuda")
    lens.map(out=out, **req)
    lens.map(out=exact, w_out=w, **req)
    assert float((out - exact).norm() / exact.norm()) < 1e-9
