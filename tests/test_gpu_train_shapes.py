"""GPU: the network's gradient and training step at ragged numbers of rows (part of
a wavefront's 32 samples, of a group of 128, and more rows than one launch takes)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _rows(n, seed):
    rng = np.random.default_rng(seed)
    X = rng.normal(0, 1.5, (n, 12)).astype(np.float32)
    return X, (X[:, 0] + X[:, 5] > 0.3).astype(np.uint8)


def _bf16(a):
    u = np.asarray(a, np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)


# (tolerances: bf16 rounding of weights, inputs and back-propagated gradients, 2^-9
# each, in the 2-norm of a parameter block)
@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 128, 129, 65536 + 77])
def test_gradient_equals_the_oracle(orc, n):
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    X, y = _rows(n, n)
    net = mlm.Refiner(seed=9)
    Q = mlm.params_to_dict(net.params)
    for k in ("W1", "W2", "W3"):
        Q[k] = _bf16(Q[k])
    ref, G = orc.mlp_loss_grad(Q, _bf16(X), y, pos_weight=2.0)
    loss, g = net.grads(X, y, pos_weight=2.0)
    gd = mlm.params_to_dict(g)
    assert abs(loss - ref) < 2.0 ** -8 * abs(ref) + 1e-6
    for k in G:
        assert np.linalg.norm(gd[k] - G[k]) < 2.0 ** -6 * np.linalg.norm(G[k]) + 1e-7, k


@pytest.mark.parametrize("n,batch", [(33, 33), (300, 300), (65536 + 77, 70000)])
def test_first_step_is_adams(n, batch):
    import torch
    import paper_2506_02114_amd as mlm
    torch.cuda.init()
    X, y = _rows(n, 5)
    net = mlm.Refiner(seed=9)
    p0 = net.params.copy()
    _, g = net.grads(X, y, pos_weight=1.0)
    for graph in (True, False):
        net = mlm.Refiner(p0)
        net.train(X, y, epochs=1, batch=batch, lr=1e-3, pos_weight=1.0, seed=1, graph=graph)
        # the first step is lr g / (|g| + 1e-8); rows in another order change g by rounding
        sure = np.abs(g) > 1e-4
        assert np.abs(net.params - p0 + 1e-3 * np.sign(g))[sure].max() < 2e-6
        # and the kernels' copies of the weights follow: the logits are the new ones
        assert np.array_equal(net.predict(X[:64]), mlm.Refiner(net.params).predict(X[:64]))
