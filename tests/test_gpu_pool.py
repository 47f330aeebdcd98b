"""GPU: device blocks pass from one lens to the next.  Maps of lenses made,
mapped and closed one after the other, of growing and shrinking size, on two
streams and from two threads, equal the same maps of lenses that stay open."""
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [(300, 96), (3000, 200), (50, 33), (800, 150), (3000, 64), (1, 40)]


def _lens(n):
    import paper_2506_02114_amd as mlm
    sf = W.star_field(n, 0.3, "salpeter", seed=n)
    return mlm.Lens(0.3, 0.05, 0.2, sf.x, sf.y, sf.m)


def _map(lens, px, out):
    return lens.map(out=out, hw1=2.0, hw2=2.0, n1=px, n2=px, rays_per_pixel=2.0)[0]


def test_blocks_move_between_lenses_streams_and_threads():
    import torch
    torch.cuda.init()
    kept = [_lens(n) for n, _ in SIZES]
    ref = [_map(l, px, torch.empty((px, px), dtype=torch.float64, device="cuda")).clone()
           for l, (_, px) in zip(kept, SIZES)]
    torch.cuda.synchronize()
    bad = []

    def work(shift):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for k in range(3 * len(SIZES)):
                i = (k * (1 + shift) + shift) % len(SIZES)
                n, px = SIZES[i]
                lens = _lens(n)
                got = _map(lens, px, torch.empty((px, px), dtype=torch.float64, device="cuda"))
                lens.close()
                st.synchronize()
                # sums of a few hundred deposits of like sign in varying order
                if not torch.allclose(got, ref[i], rtol=1e-12, atol=0):
                    bad.append((shift, k, i))

    threads = [threading.Thread(target=work, args=(s,)) for s in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    for l in kept:
        l.close()


def test_a_refiner_after_lenses_starts_from_its_own_buffers():
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    f = np.random.default_rng(3).standard_normal((5000, 12)).astype(np.float32)
    y = (f[:, 0] > 0).astype(np.uint8)
    out = []
    for _ in range(3):
        lens = _lens(500)
        _map(lens, 64, torch.empty((64, 64), dtype=torch.float64, device="cuda"))
        lens.close()
        net = mlm.Refiner(seed=5)
        losses = net.train(f, y, epochs=2, batch=512)
        out.append((losses, net.params))
        net.close()
    for losses, params in out[1:]:   # training is the same bits every time
        assert np.array_equal(losses, out[0][0]) and np.array_equal(params, out[0][1])
