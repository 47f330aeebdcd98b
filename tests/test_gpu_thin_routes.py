"""GPU: thin cells beside a threshold, with the large triangles listed and with the
lists overflowing.

No star and an almost singular lens (lambda_2 = 1e-7): every cell is a sliver along
u, 2e-8 to 2e-6 pixels thick, every second column of vertices lies on a line between
pixels but for rounding, and triangles of two pixels are large ones.  Shot by
patches and ray by ray a vertex falls to different sides of its line, so a pass that
takes a cell for large by other vertices than the pass that apportioned it counts
it twice or drops it.

Every ray lies in the map, so the map's pixels are sums of whole cells: as many
weights as cells in all; each pixel column holds two cells a row, up to the share
beyond a line of a cell of half a pixel, 1e-13.  Long sums of up to 600 like
deposits: 1e-11 relative.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,overflow", [(181, False), (301, True), (601, True)])
@pytest.mark.parametrize("big", [1, 0])
def test_cells_on_pixel_lines_count_once(nr, overflow, big):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    gamma = 0.5
    lens = mlm.Lens(0.0, 0.5 - 1e-7, gamma, np.zeros(0), np.zeros(0), np.zeros(0), sheet="none")
    lam1 = 1.0 - (0.5 - 1e-7) + gamma
    n1 = (nr - 1) // 2
    # (n2 odd: the slivers lie in the middle row of pixels; fewer than 64 cells a pixel)
    req = dict(hw1=lam1 * 1.3, hw2=1.0, n1=n1, n2=51, nray1=nr, nray2=nr, dx1=1.3, dx2=1.0, big_pixels=big)
    mu, st = lens.map(**req)
    ref, sr = lens.map(noalloc=True, **req)   # ray by ray
    assert st["n_tiles"] < sr["n_tiles"] / 2   # by patches there, by tiles of 64 rays here
    cells = (nr - 1) ** 2
    if big:
        # more than the lists' entries, or less than half of them
        cap = 64 * max(1024, (cells // 4 + 63) // 64)
        assert st["n_big"] > cap if overflow else 0 < st["n_big"] < cap
    R = lens.region(**req)
    weight = R["d1"] * R["d2"] / (R["pix1"] * R["pix2"])
    for m in (mu, ref):
        assert abs(m.sum() / (cells * weight) - 1) < 1e-11
        assert np.abs(m[25] / (2 * (nr - 1) * weight) - 1).max() < 1e-11
