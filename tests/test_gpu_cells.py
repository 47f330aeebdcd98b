"""GPU: the cell pass for maps of many cells per pixel (k_ipm_fine, with its
48-pixel window from 64 cells a pixel and its 24-pixel one from 400) and the lists
of large triangles, against the oracle's clipping of every triangle.

Positions come from the library itself, so only the apportioning is compared:
each pixel sums at most a few thousand deposits whose pixel areas are rounded to
a few units of the last place of the cell's coordinates (below 100 pixels,
1.4e-14, over cells at least 1e-4 pixels wide): 1e-9 relative with margin.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,nr1,nr2,gamma", [
    (16, 16, 131, 165, 0.1),      # 84 cells a pixel; tiles of 32 x 32 cells, 130 columns and 164 rows
    (16, 12, 129, 129, -0.35),    # elongated the other way
    (8, 8, 201, 185, 0.1),        # 575 cells a pixel
    (5, 9, 257, 97, 0.55),        # 546, elongated, one tile row and a row over
    (8, 8, 180, 33, 0.2),         # 90, a single tile row
    (40, 40, 65, 66, 0.3),        # 2.6: the pass for ordinary maps
    (8, 8, 161, 162, 0.4),        # with large triangles only (see big_pixels)
])
@pytest.mark.parametrize("big", [0, 2])
def test_map_equals_clipping(orc, n1, n2, nr1, nr2, gamma, big):
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    sf = W.star_field(30, 0.3, "salpeter", seed=21)
    spec = dict(hw1=1.1, hw2=0.9, n1=n1, n2=n2, nray1=nr1, nray2=nr2, order=16)
    gl = mlm.Lens(0.3, 0.05, gamma, sf.x, sf.y, sf.m)
    mu, st = gl.map(big_pixels=big, **spec)
    ref = orc.magnification_map(orc.Lens(0.3, 0.05, gamma, sf.x, sf.y, sf.m), spec, method="fmm", p=16)
    assert st["n_big"] > 0 if big else True
    pos = ref.mu > 1e-6
    assert np.abs(mu[pos] / ref.mu[pos] - 1).max() < 1e-9
    assert np.abs(mu[~pos] - ref.mu[~pos]).max(initial=0.0) < 1e-10
