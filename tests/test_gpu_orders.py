"""FMM coefficients over the expansion orders (rounds of loads and of orders with
remainders of every length) against the oracle's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 8, 9, 11, 16, 17, 20, 25, 31])
def test_coefficients_equal_the_oracle(orc, p):
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    rng = np.random.default_rng(p)
    n = 700
    # a knot of stars in a thin field: leaves of several levels next to each other
    x, y = np.concatenate([rng.uniform(-5, 5, (2, n - 300)), 1.3 + 0.1 * rng.standard_normal((2, 300))], 1)
    m = rng.uniform(0.1, 1.0, n)
    ex = mlm.Lens(0.3, 0.0, 0.1, x, y, m).fmm_export(hw1=2.0, hw2=2.0, n1=16, n2=16, nray1=9, nray2=9, order=p)
    F = orc.FMM(orc.Lens(0.3, 0.0, 0.1, x, y, m), ex["info"]["L0"], p)
    nd = F.nodes()
    ro = np.lexsort((nd["j"], nd["i"], nd["level"]))
    go = np.lexsort((ex["j"], ex["i"], ex["level"]))
    oa, oc = F.coeffs()
    # sums of some thousand terms of both signs, to the rounding of the largest
    for g, o in ((ex["mult"][go], oa[ro]), (ex["local"][go][:, 1:], oc[ro][:, 1:])):
        assert (np.abs(g - o) <= 1e-11 * np.maximum(np.abs(o).max(axis=1, keepdims=True), 1e-300)).all()
