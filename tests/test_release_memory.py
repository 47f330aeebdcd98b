"""The library's pool of idle blocks: bounded, emptied by age and on request."""
import numpy as np
import pytest

import workloads as W


def test_nothing_to_release_without_a_lens():
    import subprocess
    import sys
    code = "import paper_2506_02114_amd as m; assert m.release_memory() == 0"
    subprocess.run([sys.executable, "-c", code], check=True)


def _mlm():
    import torch   # before the library: both then share one HIP runtime
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    mlm.release_memory()
    return torch, mlm


def _lens(mlm, n=300):
    sf = W.star_field(n, 0.3, "salpeter", seed=n)
    return mlm.Lens(0.3, 0.05, 0.2, sf.x, sf.y, sf.m)


MAP = dict(hw1=2.0, hw2=2.0, n1=64, n2=64, nray1=4000, nray2=3000)   # 192 MB of vertices


@pytest.mark.gpu
def test_release_gives_the_device_its_memory_back():
    torch, mlm = _mlm()
    lens = _lens(mlm)
    mu, _ = lens.map(**MAP)
    held = lens.map(**MAP)[0]
    lens.close()
    free0 = torch.cuda.mem_get_info()[0]
    got = mlm.release_memory()
    assert got >= 8 * 2 * MAP["nray1"] * MAP["nray2"]
    # (the runtime may keep what it cut into small blocks)
    assert torch.cuda.mem_get_info()[0] - free0 > 0.9 * got
    assert mlm.release_memory() == 0
    again = _lens(mlm).map(**MAP)[0]
    assert np.allclose(again, mu, rtol=1e-12, atol=0) and np.allclose(held, mu, rtol=1e-12, atol=0)


@pytest.mark.gpu
def test_blocks_age_as_lenses_come_and_go():
    torch, mlm = _mlm()
    lens = _lens(mlm)
    lens.map(**MAP)
    lens.close()
    for _ in range(70):   # small lenses that take none of the large blocks
        _lens(mlm, 1).close()
    assert mlm.release_memory() < 8 * 2 * MAP["nray1"] * MAP["nray2"]


@pytest.mark.gpu
def test_at_most_four_gib_are_kept():
    torch, mlm = _mlm()
    req = dict(MAP, nray1=9000, nray2=8000)   # a strip of 1 GiB each
    lenses = [_lens(mlm, 50 + k) for k in range(6)]
    for lens in lenses:
        lens.map(**req)
    for lens in lenses:
        lens.close()
    assert 2 << 30 < mlm.release_memory() <= 4 << 30


@pytest.mark.gpu
def test_release_beside_maps_of_other_threads():
    import threading
    torch, mlm = _mlm()
    ref, _ = _lens(mlm).map(hw1=2.0, hw2=2.0, n1=64, n2=64, rays_per_pixel=4.0)
    bad, stop = [], threading.Event()

    def work():
        for _ in range(20):
            lens = _lens(mlm)
            mu, _ = lens.map(hw1=2.0, hw2=2.0, n1=64, n2=64, rays_per_pixel=4.0)
            lens.close()
            if not np.allclose(mu, ref, rtol=1e-12, atol=0):
                bad.append(mu)
        stop.set()

    t = threading.Thread(target=work)
    t.start()
    while not stop.wait(0.002):
        mlm.release_memory()
    t.join()
    assert not bad
