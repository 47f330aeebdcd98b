"""GPU: which cells the learned refinement takes, at the ends of its threshold: every
cell (then the map is the plain refinement's), or the folded ones alone, counted
here from the rays' positions by the same signs of the same products."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# grids narrower than the 64 cells that are flagged together, of a whole number of
# them, and with a remainder
@pytest.mark.parametrize("nr1,nr2", [(2, 90), (20, 211), (65, 65), (130, 47), (33, 3)])
def test_flagged_cells(nr1, nr2):
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    sf = W.star_field(60, 0.4, "salpeter", seed=4)
    lens = mlm.Lens(0.4, 0.0, 0.2, sf.x, sf.y, sf.m)
    spec = dict(hw1=1.2, hw2=1.0, n1=24, n2=20, nray1=nr1, nray2=nr2, order=14)
    rf = dict(refine_depth=2, refine_window=6)
    net = mlm.Refiner(seed=2)
    plain, sp = lens.map(refine="plain", **spec, **rf)
    every, se = lens.map(refine="learned", refiner=net, refine_threshold=-1e30, **spec, **rf)
    ncells = (nr1 - 1) * (nr2 - 1)
    assert se["n_refine_candidates"] == sp["n_refine_candidates"] == ncells
    assert se["n_refined"] == sp["n_refined"]
    assert np.abs(every - plain).max() <= 1e-12 * np.abs(plain).max()    # (another order of the same deposits)
    w = np.zeros((nr2, nr1, 2))
    lens.map(w_out=w, **spec)
    # pixel coordinates as the library forms them, up to rounding, which no ear here is near enough to feel
    u = (w[..., 0] + 1.2) / (2.4 / 24)
    v = (w[..., 1] + 1.0) / (2.0 / 20)
    q = [(u[j0:nr2 - 1 + j0, i0:nr1 - 1 + i0], v[j0:nr2 - 1 + j0, i0:nr1 - 1 + i0])
         for i0, j0 in ((0, 0), (1, 0), (1, 1), (0, 1))]
    s = []
    for k in range(4):
        (ua, va), (ub, vb), (uc, vc) = q[k], q[(k + 1) % 4], q[(k + 3) % 4]
        s.append(np.sign((ub - ua) * (vc - va) - (uc - ua) * (vb - va)))
    folded = int((~((s[0] == s[1]) & (s[1] == s[2]) & (s[2] == s[3]))).sum())
    _, sf_ = lens.map(refine="learned", refiner=net, refine_threshold=1e30, **spec, **rf)
    assert sf_["n_refine_candidates"] == folded
