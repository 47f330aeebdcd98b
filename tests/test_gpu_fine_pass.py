"""GPU: k_ipm_fine, the cell pass of strips of at least 4e6 cells on maps of at least
64 cells a pixel, against k_ipm, which maps without allocation take (their strips are
smaller), and once against the oracle's clipping of every triangle.

Rays are shot one by one on both sides, so only the apportioning is compared: pixel
areas are rounded to a few units of the last place of the coordinates (below 200
pixels, 2.8e-14, over cells at least 1e-2 pixels wide; a pixel holds hundreds of
them): 1e-9 relative with margin.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = {
    # name: (pixels, rays)
    "whole_tiles": ((200, 200), (2049, 2049)),       # 105 cells a pixel; 2048 x 2048 cells
    "remainders": ((200, 150), (2050, 2080)),        # 142; 2049 columns, 2079 rows
    "small_window": ((60, 60), (2111, 2011)),        # 1178: the 24-pixel window
    "long_rows": ((50, 80), (8193, 545)),            # 1114, elongated cells
    "long_columns": ((150, 150), (513, 9001)),       # 205, elongated the other way
    "narrow_map": ((3, 70), (2049, 2100)),
}


def _setup(name):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    px, rays = CASES[name]
    sf = W.star_field(30, 0.3, "salpeter", seed=21)
    spec = dict(hw1=1.1, hw2=0.9, n1=px[0], n2=px[1], nray1=rays[0], nray2=rays[1], order=16)
    return torch, mlm.Lens(0.3, 0.05, 0.1, sf.x, sf.y, sf.m), spec, sf


def _map(torch, lens, spec, **kw):
    out = torch.empty((spec["n2"], spec["n1"]), dtype=torch.float64, device="cuda")
    w = torch.empty((spec["nray2"], spec["nray1"], 2), dtype=torch.float64, device="cuda")
    lens.map(out=out, w_out=w, **spec, **kw)
    return out


def _close(mu, ref):
    pos = ref > 1e-6
    assert float((mu[pos] / ref[pos] - 1).abs().max()) < 1e-9
    assert float((mu - ref)[~pos].abs().sum()) < 1e-10


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("big", [0, 2, 4])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_map_equals_the_ordinary_pass(name, big, precision):
    torch, lens, spec, _ = _setup(name)
    mu = _map(torch, lens, spec, big_pixels=big, precision=precision)
    ref = torch.empty_like(mu)
    _, st = lens.map(out=ref, noalloc=True, big_pixels=big, precision=precision, **spec)
    assert st["n_ipm_launches"] > 1   # strips below 4e6 cells
    _close(mu, ref)


def test_map_equals_clipping(orc):
    torch, lens, spec, sf = _setup("remainders")
    mu = _map(torch, lens, spec)
    ref = orc.magnification_map(orc.Lens(0.3, 0.05, 0.1, sf.x, sf.y, sf.m), spec, method="fmm", p=16)
    _close(mu, torch.from_numpy(ref.mu).cuda())
