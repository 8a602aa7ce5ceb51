"""The warm-start network over the shapes where its kernels divide work
differently: widths off every tile, layers too wide for the chain kernel,
batches on both sides of the sample blocks (16, 32) and of the rules that give
a workgroup more of them, and batches smaller than the one before."""
import numpy as np
import pytest

import workloads as W
from oracle import mlp as ref

pytestmark = pytest.mark.gpu

WIDE = (2, 1200, 33, 900)          # layers past the chain's LDS: one launch per product
SHAPES = [(1, 2), (3, 31, 32, 33), (17, 64, 1, 100, 64), (64, 992, 992), (5, 1000, 7), WIDE]


@pytest.fixture(scope="module")
def P():
    import paper_2609_17151_amd as P
    return P


def _bf16(a):
    """Round to the nearest BF16 (ties to even), as float64."""
    u = np.asarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32).view(np.float32).astype(np.float64)


def _reference(p, widths, x, t):
    """Outputs, loss and gradient with every product's operands rounded to
    BF16, as the network is defined, and FP64 sums."""
    layers = ref.split(np.asarray(p, np.float64), widths)
    ones = np.ones((len(x), 1))
    a, zs, ins = x.astype(np.float64), [], []
    for i, w in enumerate(layers):
        ins.append(np.hstack([_bf16(a), ones]))
        z = ins[-1] @ _bf16(w).T
        zs.append(z)
        a = ref.gelu(z) if i + 1 < len(layers) else z
    y, d = zs[-1], zs[-1] - t.astype(np.float32)
    dz, grads = 2.0 * d / d.size, [None] * len(layers)
    for i in reversed(range(len(layers))):
        grads[i] = _bf16(dz).T @ ins[i]
        if i:
            dz = (_bf16(dz) @ _bf16(layers[i])[:, :-1]) * ref.gelu_grad(zs[i - 1])
    return y, float(np.mean(d * d)), np.concatenate([g.ravel() for g in grads])


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("widths", SHAPES)
@pytest.mark.parametrize("batch", [1, 16, 33, 97])
def test_shapes_match_reference(P, widths, batch):
    # the network tests' 2e-2 on outputs and gradients, against products of the
    # same BF16 operands: a layer one unit wide has no average over roundings
    p = (W.mlp_init(widths, seed=5) + 0.01).astype(np.float32)
    x, t = W.mlp_batch(batch, widths[0], widths[-1], seed=batch)
    net = P.MLP(widths, max_batch=batch)
    net.set_params(p)
    p64 = p.astype(np.float64)
    y_ref, loss_ref, g_ref = _reference(p64, widths, x.astype(np.float32), t)
    y = net.forward(x).cpu().numpy()
    loss, g = net.grad(x, t)
    assert _rel(y, y_ref) <= 2e-2
    assert loss == pytest.approx(loss_ref, rel=2e-2)
    assert _rel(g.astype(np.float64), g_ref) <= 2e-2
    # the update follows the same gradient: Adam's first step in FP32
    net.train_step(x, t, lr=1e-3)
    g64 = g.astype(np.float64)
    expect = p64 - 1e-3 * g64 / (np.abs(g64) + 1e-8)
    assert np.abs(net.params() - expect).max() <= 1e-6 * 1e-3 + 2e-7 * np.abs(p).max()
    # and the products then read the updated weights
    y1_ref = _reference(net.params(), widths, x.astype(np.float32), t)[0]
    assert _rel(net.forward(x).cpu().numpy(), y1_ref) <= 2e-2
    net.close()


@pytest.mark.parametrize("widths", [(5, 64, 64, 48), WIDE])
def test_a_sample_does_not_depend_on_its_batch(P, widths):
    # rows per workgroup and kernel follow the batch; every row's sums keep
    # their order, so its outputs are the same bits in any batch
    n = 17000
    x, _ = W.mlp_batch(n, widths[0], widths[-1], seed=9)
    net = P.MLP(widths, max_batch=n)
    net.set_params(W.mlp_init(widths, seed=6) + 0.01)
    y = net.forward(x).cpu().numpy()
    for m in (1, 15, 17, 4096, 4097, 8193):
        assert np.array_equal(net.forward(x[:m]).cpu().numpy(), y[:m]), m
    net.close()


@pytest.mark.parametrize("widths", [(5, 64, 64, 48), WIDE])
def test_gradient_of_a_small_batch_after_a_large_one(P, widths):
    # the rows a larger batch left in the workspaces take no part
    x, t = W.mlp_batch(8209, widths[0], widths[-1], seed=10)
    p = W.mlp_init(widths, seed=7) + 0.01
    used, fresh = P.MLP(widths, max_batch=8209), P.MLP(widths, max_batch=64)
    used.set_params(p)
    fresh.set_params(p)
    used.grad(x, t)
    for m in (64, 37, 1):
        la, ga = used.grad(x[:m], t[:m])
        lb, gb = fresh.grad(x[:m], t[:m])
        assert la == lb and np.array_equal(ga, gb), m
    # the gradient of all rows is the mean of the parts', to FP32 sums
    _, g = used.grad(x, t)
    cut = 4100
    _, g1 = used.grad(x[:cut], t[:cut])
    _, g2 = used.grad(x[cut:], t[cut:])
    part = (g1.astype(np.float64) * cut + g2.astype(np.float64) * (len(x) - cut)) / len(x)
    assert _rel(g.astype(np.float64), part) <= 1e-2
    used.close()
    fresh.close()
