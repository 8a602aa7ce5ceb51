"""The warm-start network on both sides of the rules that choose its kernels by
widths and batch: a sample's outputs do not depend on which kernel formed them,
and gradients match the products of the same BF16 operands."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_mlp_shapes import _reference, _rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_17151_amd as P
    return P


def _net(P, widths, batch, seed=5):
    net = P.MLP(widths, max_batch=batch)
    p = (W.mlp_init(widths, seed=seed) + 0.01).astype(np.float32)
    net.set_params(p)
    return net, p


@pytest.mark.parametrize("widths,batches", [
    # 66 tiles across the first layer's padded rows, 64 across the outputs: 4096
    # tiles are passed from 960 to 1009 samples (padded to 1024) and from 1024 to 1025
    ((7, 1024, 1024), (64, 960, 1009, 1024, 1025, 1088)),
    # 76 across: 3952 tiles at 832 samples, 4256 at 833 (padded to 896)
    ((3, 1200, 1210), (800, 832, 833)),
])
def test_tiles_of_a_wave_and_of_a_workgroup(P, widths, batches):
    n = max(batches)
    x, t = W.mlp_batch(n, widths[0], widths[-1], seed=3)
    net, p = _net(P, widths, n)
    y = net.forward(x).cpu().numpy()
    for m in batches:
        assert np.array_equal(net.forward(x[:m]).cpu().numpy(), y[:m]), m
        y_ref, loss_ref, g_ref = _reference(p, widths, x[:m].astype(np.float32), t[:m])
        loss, g = net.grad(x[:m], t[:m])
        assert _rel(y[:m], y_ref) <= 2e-2
        assert loss == pytest.approx(loss_ref, rel=2e-2)
        assert _rel(g.astype(np.float64), g_ref) <= 2e-2
    net.close()


@pytest.mark.parametrize("widths", [(5, 448, 448, 448, 768), (5, 512, 512, 512, 768), (900, 900), (3, 31, 940, 700, 33)])
@pytest.mark.parametrize("max_batch", [40, 800])
def test_the_chain_and_a_launch_per_product(P, widths, max_batch):
    # networks of more than 0.42 MB of weights per product take a launch per
    # product up to 256 samples (0.6 MB: 768), the chain above.  448 wide:
    # prediction by the chain, training of few samples by a launch per product;
    # (900, 900) is past 0.6 MB
    x, t = W.mlp_batch(max_batch, widths[0], widths[-1], seed=4)
    net, p = _net(P, widths, max_batch)
    y = net.forward(x).cpu().numpy()
    for m in (1, 40, 256, 257, 768, 769):
        if m > max_batch:
            continue
        assert np.array_equal(net.forward(x[:m]).cpu().numpy(), y[:m]), m
        y_ref, loss_ref, g_ref = _reference(p, widths, x[:m].astype(np.float32), t[:m])
        loss, g = net.grad(x[:m], t[:m])
        assert _rel(y[:m], y_ref) <= 2e-2
        assert loss == pytest.approx(loss_ref, rel=2e-2)
        assert _rel(g.astype(np.float64), g_ref) <= 2e-2
        g64, before = g.astype(np.float64), net.params().astype(np.float64)
        net.set_params(p)                               # clears the moments
        net.train_step(x[:m], t[:m], lr=1e-3)
        expect = before - 1e-3 * g64 / (np.abs(g64) + 1e-8)
        assert np.abs(net.params() - expect).max() <= 1e-6 * 1e-3 + 2e-7 * np.abs(p).max()
        net.set_params(p)
    net.close()


def test_more_input_elements_than_a_launch_has_threads(P):
    # 2^20 samples (the most a network takes) of 4096 inputs and their ones are
    # more than 2^32 elements; the last rows give the same bits on their own
    n, widths = 1 << 20, (4096, 3)
    net, _ = _net(P, widths, n)
    x = torch.randn((n, widths[0]), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    y = net.forward(x)
    for at in (0, n // 2 - 20, n - 40):
        assert bool(torch.equal(y[at:at + 40], net.forward(x[at:at + 40]))), at
    net.close()
    del x, y
    torch.cuda.empty_cache()
