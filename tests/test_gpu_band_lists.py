"""GPU: the band lists of millions of large triangles, sorted in LDS, against the
batch's, whose entries go to their lists one by one.

Both apportion the same rays in mixed precision (shot ray by ray in both) by the
same arithmetic; only the order of a pixel's FP64 sums differs.  A pixel sums up to
~1e4 deposits and column differences of either sign, each no larger than the
brightest pixel: 1e4 roundings of 1.1e-16 of it, 1.1e-12 of the map's largest value.
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = {
    # short triangles, most workgroups sort; long and short ones, some write directly
    "many_stars": (W.star_field, (100_000, 0.45, "kroupa"), (0.45, 0.0, 0.45), 25.0),
    "elongated_cells": (W.star_field, (26_730, 0.6, "equal"), (0.6, 0.0, 0.6), 10.0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_sorted_lists_equal_the_batch(name):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    field, args, (ks, kss, gamma), hw = CASES[name]
    sf = field(*args, seed=5)
    lens = mlm.Lens(ks, kss, gamma, sf.x, sf.y, sf.m)
    req = dict(hw1=hw, hw2=hw, n1=2000, n2=2000, precision="mixed")
    out = torch.empty((2000, 2000), dtype=torch.float64, device="cuda")
    ref = torch.empty_like(out)
    _, st = lens.map(out=out, timing=2, **req)
    assert st["n_band_rows"] >= 4 << 24   # bands of four rows: at least 2^24 entries
    mlm.map_batch([lens], [req], [ref])
    assert float(ref.max()) > 0
    assert float((out - ref).abs().max() / ref.max()) < 1.1e-12
