"""The warm-start network on both sides of the rules that choose its kernels by
widths and batch: a sample's outputs do not depend on which kernel formed them,
and gradients match the products of the same BF16 operands."""
import numpy as np
import pytest

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
    # layers of 1024 outputs, 64 tiles of 16 across: 4096 tiles at 1024 samples
    ((7, 1024, 1024), (64, 1009, 1024, 1025, 1088)),
    # the last layer's padded row of 1216, 76 across: 4104 tiles at 864 samples
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
