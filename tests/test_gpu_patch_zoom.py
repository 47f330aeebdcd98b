"""GPU: ray shooting by patches on maps whose pixels are small against the
positions: down to 1e-11 of them, where a position's rounding is 1e-5 pixels and
more.  Counts have to be those of shooting ray by ray; below that the map is shot
ray by ray."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("at", [(4.1, -2.3), (0.3, 0.2)])
@pytest.mark.parametrize("nr", [401, 2201, 6001])   # patches of 32 and of 64 rays
@pytest.mark.parametrize("pix,patches", [(1e-6, True), (1e-8, True), (1e-9, True), (1e-10, True), (1e-13, False)])
def test_counts_equal_ray_by_ray(pix, patches, nr, at):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    sf = W.star_field(40, 0.3, "salpeter", seed=13)
    lens = mlm.Lens(0.3, 0.1, 0.25, sf.x, sf.y, sf.m)
    n = 50
    req = dict(n1=n, n2=n, order=18)
    y = lens.deflect(np.array([at]), hw1=1.0, hw2=1.0, **req)[0]
    # the map about the point's image, filled by the rays about the point
    req.update(y1c=y[0], y2c=y[1], hw1=0.5 * n * pix, hw2=0.5 * n * pix, x1c=at[0], x2c=at[1], dx1=n * pix, dx2=n * pix,
               nray1=nr, nray2=nr - 12)
    got, st = lens.map(mapping="irs", **req)
    ref, sr = lens.map(mapping="irs", noalloc=True, **req)
    assert (st["n_tiles"] < sr["n_tiles"] / 2) == patches
    assert (ref > 0).mean() > 0.1   # the rays land in the map
    assert np.array_equal(got, ref)
