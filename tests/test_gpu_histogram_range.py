"""GPU: histograms over ranges so wide that log10 of a pixel, less the lower end,
rounds to steps as wide as the FP32 estimate's error: the counts are those of the
formula in FP64 (whole counts: exactly equal)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi", [(-1e10, 1e10), (-3e9, 1e9), (-1e12, 3e12), (-1e8, 1e8), (-4.0, 3.0)])
@pytest.mark.parametrize("bins", [8000, 1000])
def test_bins_equal_the_formula(lo, hi, bins):
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    inv = bins / (hi - lo)
    # pixels around the edges within the doubles' range, closer than such a step
    edges = lo + (hi - lo) / bins * np.arange(bins + 1)
    edges = edges[np.abs(edges) < 300][:50]
    step = max(np.spacing(abs(lo)), 1e-7)
    x = torch.tensor((edges[:, None] + 4 * step * np.linspace(-1, 1, 20001)).ravel(), device="cuda")
    m = 10.0 ** torch.clamp(x, -300, 300)
    b = 1 + torch.floor((torch.log10(m) - lo) * inv)
    b = torch.clamp(b, 0, bins + 1)
    want = torch.bincount(b.long(), minlength=bins + 2)
    got = mlm.histogram(m.view(1, -1), lo, hi, bins, hw1=1.0, hw2=1.0, n1=m.numel(), n2=1)
    assert edges.size > 0 and torch.equal(got, want)
