"""GPU: the two ways a map's large triangles go, by the lists that the cell pass
keeps (mlm_map) and counted and gathered by cell tiles (mlm_map_noalloc, and
mlm_map where a list overflows), for every cell pass and threshold of "large",
against the oracle's clipping of every triangle.  A pass that deposits a triangle
which the other way counts as large, or the reverse, loses it or counts it twice.
(The densities named fine_* take k_ipm_fine only in strips of 4e6 cells and more:
test_gpu_fine_pass.py.)

Tolerances: 1e-9 relative as in test_gpu_cells.py, whose cells are at least 1e-4
pixels thick.  The elongated cells of the overflowing lists fold to triangles
1.7e-8, 1.0e-8 and 2.5e-9 pixels thick (from the positions in 64 bits); the rounding
of a position below 64, 64 and 16 pixels, 1.4e-14 and 3.6e-15, is up to 1.4e-6 of
that, and a triangle's deposits are quotients by its area, so each pixel may be off
by a few times that, 3.6e-6, of a triangle's weight besides.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = {
    # name: (pixels, rays)
    "window_48": ((40, 40), (65, 66)),            # 2.6 cells a pixel
    "window_32": ((20, 20), (131, 117)),          # 38
    "fine_48": ((16, 16), (131, 165)),            # 84
    "fine_24": ((6, 6), (201, 185)),              # 1022
}
OVERFLOW = {   # all rays inside the map, the cells of the last three several pixels long
    "window_48": ((300, 300), (401, 397)),        # 1.8 cells a pixel
    "window_32": ((64, 64), (11, 16001)),         # 39
    "fine_48": ((64, 64), (11, 30001)),           # 73
    "fine_24": ((16, 16), (5, 60001)),            # 938
}


def _pair(orc, px, rays, gamma=0.1, **kw):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    sf = W.star_field(30, 0.3, "salpeter", seed=21)
    spec = dict(hw1=1.1, hw2=0.9, n1=px[0], n2=px[1], nray1=rays[0], nray2=rays[1], order=16, **kw)
    ref = orc.magnification_map(orc.Lens(0.3, 0.05, gamma, sf.x, sf.y, sf.m), spec, method="fmm", p=16)
    return mlm.Lens(0.3, 0.05, gamma, sf.x, sf.y, sf.m), spec, ref.mu


def _close(mu, ref, thin=0.0):
    assert np.all(np.abs(mu - ref) < 1e-9 * ref + np.where(ref > 1e-6, 0.0, 1e-10) + thin)


@pytest.mark.parametrize("name", list(GRIDS))
@pytest.mark.parametrize("big", [1, 2, 4, 0])
def test_lists_and_tiles_equal_clipping(orc, name, big):
    gl, spec, ref = _pair(orc, *GRIDS[name])
    for noalloc in (False, True):
        mu, st = gl.map(noalloc=noalloc, big_pixels=big, **spec)
        assert st["n_big"] > 0 if big else True
        _close(mu, ref)


@pytest.mark.parametrize("name", list(OVERFLOW))
@pytest.mark.parametrize("big", [1, 2])
def test_overflowing_lists_equal_clipping(orc, name, big):
    gl, spec, ref = _pair(orc, *OVERFLOW[name], dx1=1.0, dx2=1.0)
    mu, st = gl.map(big_pixels=big, **spec)
    # more than the lists' 64 x max(1024, cells / 256) entries
    assert st["n_big"] > 64 * max(1024, (st["n_cells"] // 4 + 63) // 64)
    R = gl.region(**spec)
    _close(mu, ref, 3.6e-6 * 0.5 * R["d1"] * R["d2"] / (R["pix1"] * R["pix2"]))
