"""GPU: maps whose large triangles do not fit the scratch array beside a vertex strip
of a quarter of it: they are made by strips of an eighth, and equal mlm_map's to the
rounding of the sums' order (1e-12 relative, as in test_zz_no_alloc.py) and of
slivers, whose deposits' terms are larger than the deposits by the cell's extent over
the sliver's thickness: 4 units in the last place of the pixel coordinates over the
thickness of the thinnest triangle that crosses a pixel line, of a triangle's weight."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,req", [
    (8000, dict(hw1=5.0, hw2=5.0, n1=1000, n2=1000, rays_per_pixel=1.0)),
    (4500, dict(hw1=5.0, hw2=5.0, n1=600, n2=600, rays_per_pixel=2.0, order=31)),
])
def test_map_equals_the_allocating_one(n, req):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    sf = W.star_field(n, 0.4, "salpeter", seed=3)
    lens = mlm.Lens(0.4, 0.1, 0.2, sf.x, sf.y, sf.m)
    out = torch.empty((req["n2"], req["n1"]), dtype=torch.float64, device="cuda")
    ref = torch.empty_like(out)
    w = torch.empty((lambda R: (R["nr2"], R["nr1"], 2))(lens.region(**req)), dtype=torch.float64, device="cuda")
    lens.map(out=ref, w_out=w, **req)   # (rays one by one, as inside the array)
    _, st = lens.map(out=out, noalloc=True, **req)
    assert st["n_shoot_launches"] > 1
    R = lens.region(**req)
    p = (w + torch.tensor([req["hw1"], req["hw2"]], device="cuda")) / torch.tensor([R["pix1"], R["pix2"]], device="cuda")
    a, b, c, d = p[:-1, :-1], p[:-1, 1:], p[1:, 1:], p[1:, :-1]
    thin = 1.0
    for t in (torch.stack((a, b, c)), torch.stack((a, c, d))):
        e, f = t[1] - t[0], t[2] - t[0]
        twice = (e[..., 0] * f[..., 1] - f[..., 0] * e[..., 1]).abs()
        lo, hi = t.min(0).values, t.max(0).values
        ok = (hi > 0).all(-1) & (lo < req["n1"]).all(-1) & (lo.floor() != hi.floor()).any(-1) & (twice > 0)
        thin = min(thin, float((twice / (hi - lo).norm(dim=-1))[ok].min()))
    weight = 0.5 * R["d1"] * R["d2"] / (R["pix1"] * R["pix2"])
    assert bool((out[ref == 0] == 0).all())
    assert bool(((out - ref).abs() <= 1e-12 * ref + 4 * np.spacing(float(req["n1"])) / thin * weight).all())


def test_a_map_beyond_any_strip_is_refused():
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    sf = W.star_field(400_000, 0.4, "salpeter", seed=3)
    lens = mlm.Lens(0.4, 0.1, 0.2, sf.x, sf.y, sf.m)
    out = torch.empty((600, 600), dtype=torch.float64, device="cuda")
    with pytest.raises(mlm.MLMError, match="MLM_ERANGE"):
        lens.map(out=out, noalloc=True, hw1=5.0, hw2=5.0, n1=600, n2=600)
    lens.map(out=out, hw1=5.0, hw2=5.0, n1=600, n2=600)
    assert float(out.sum()) > 0
