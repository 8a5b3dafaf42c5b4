"""The trainer's kernels at the batch sizes where they can go wrong: blocks of
16 rows, k steps of 32, splits and column-sum chunks of 256, eight k steps at a
time, and more row blocks than workgroups (16 x 512 rows on 256 compute units),
where a workgroup takes a second one."""
import numpy as np
import pytest

import paper_1211_2205_amd as pa
from oracle import mlp
from test_gpu_closure import NP, _batch, _dev, _params, _relmax

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [7, 8, 9, 15, 16, 17, 31, 32, 33, 255, 256, 257, 287, 513, 8193, 16403])
def test_gradients_at_the_edges_of_blocks(B):
    """Against the oracle with the same operand rounding, within the bounds of
    the suite's gradient test; and, to the bit, on a trainer whose workspaces
    hold a larger batch's values."""
    p = _params(21)
    X, T = _batch(B, B)
    net = pa.MLP(B)
    net.set_params(mlp.flatten(p))
    x, t = _dev(X), _dev(T)
    y = net.forward(x).cpu().numpy().astype(np.float64)
    g, loss = net.gradients(x, t)
    Yo, co = mlp.forward(p, X, bf16=True)
    go = mlp.backward(p, co, Yo, T, bf16=True)
    assert _relmax(y, Yo) < 1e-3
    assert abs(loss - mlp.loss(Yo, T)) < 1e-4 * mlp.loss(Yo, T)
    gd = mlp.unflatten(g.astype(np.float64), *NP)
    for k in mlp.NAMES:
        assert _relmax(gd[k], go[k]) < 1e-3, (k, _relmax(gd[k], go[k]))
    used = pa.MLP(2 * B + 40)
    used.set_params(mlp.flatten(p))
    X2, T2 = _batch(B + 1, 2 * B + 40)
    used.gradients(_dev(1e3 * X2), _dev(T2))
    g2, loss2 = used.gradients(x, t)
    assert np.array_equal(g, g2) and loss == loss2
    # a step is the Adam update of that gradient
    net.train_step(x, t, 1e-3)
    used.adam_step(g, 1e-3)
    assert np.array_equal(net.params(), used.params())
    net.close()
    used.close()
