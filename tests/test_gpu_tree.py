"""The tree of few stars (one workgroup) and of many (the grid) against the
oracle's: node for node, with the same stars in them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mlm():
    import torch
    import paper_2506_02114_amd as m
    torch.cuda.init()
    m.load()
    return m


# one star; a wavefront's and a workgroup's edges; the last sorted by one
# workgroup and the first by the grid; leaves so small that the coarse levels
# outgrow the workgroup; stars on one spot (the tree's full depth)
@pytest.mark.parametrize("n,leaf_max,spot", [
    (1, 32, False), (64, 8, False), (1023, 32, False), (1025, 1, False), (4096, 16, False), (4097, 16, False),
    (9000, 2, False), (40000, 32, False), (300, 32, True),
])
def test_tree_equals_the_oracle(mlm, orc, n, leaf_max, spot):
    rng = np.random.default_rng(n)
    x, y = rng.uniform(-6, 6, (2, n)) if not spot else np.full((2, n), 1.234567) + rng.uniform(-1, 1, (2, n)) * 1e-5
    m = rng.uniform(0.1, 1.0, n)
    gl = mlm.Lens(0.3, 0.0, 0.1, x, y, m)
    spec = dict(hw1=2.0, hw2=2.0, n1=16, n2=16, nray1=21, nray2=17, order=6)
    ex = gl.fmm_export(leaf_max=leaf_max, **spec)
    F = orc.FMM(orc.Lens(0.3, 0.0, 0.1, x, y, m), ex["info"]["L0"], 6, nmax=leaf_max)
    nd = F.nodes()
    ref = np.stack([nd[k] for k in ("level", "i", "j", "leaf", "nstars", "block")])
    got = np.stack([ex[k] for k in ("level", "i", "j", "leaf", "nstars", "block")])
    ro, go = np.lexsort(ref[2::-1]), np.lexsort(got[2::-1])
    assert np.array_equal(ref[:, ro], got[:, go])
    # the same stars in the same leaves: coefficients to the rounding of sums of n terms
    oa, oc = F.coeffs()
    for g, o in ((ex["mult"][go], oa[ro]), (ex["local"][go][:, 1:], oc[ro][:, 1:])):
        assert (np.abs(g - o) <= 1e-11 * np.maximum(np.abs(o).max(axis=1, keepdims=True), 1e-300)).all()
