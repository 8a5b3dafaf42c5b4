"""The closure network's kernel (blocks of 16 points per wave, 16 waves per
workgroup) at the grid sizes where it can go wrong, against the kernel that
evaluates the network inside the odd sweep: other blocks, the same operations,
so the states agree to the bit."""
import numpy as np
import pytest

import paper_1211_2205_amd as pa
import workloads as wl
from oracle import mlp
from test_gpu_closure import _params, _state_problem

pytestmark = pytest.mark.gpu

P, X = wl.BC_PERIODIC, wl.BC_EXTRAPOLATION


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,bc", [
    ((2, 2), (X, X)),      # one partial block
    ((15, 3), (P, X)),     # 64 evaluation points: whole blocks only
    ((16, 14), (X, P)),    # 255: one point short
    ((15, 15), (P, P)),    # 256
    ((256, 1 + 1), (X, X)),
    ((70, 58), (P, X)),    # about one block per workgroup
    ((255, 255), (X, X)),  # one block per wave
    ((256, 257), (X, P)),  # some waves take a second block
    ((401, 330), (P, P)),  # all do
])
def test_network_kernel_equals_the_fused_one(precision, n, bc):
    prob = _state_problem(5, n, bc, 51, precision=precision)
    p = mlp.flatten(_params(16, out_scale=0.2))
    runs = []
    for fused in (False, True):
        s = pa.Solver.from_problem(prob, precision=precision, closure="learned")
        s.load_closure(p)
        s.set_closure_fused(fused)
        s.advance(2)
        runs.append(s.moments())
        s.close()
    for k, (a, b) in enumerate(zip(*runs)):
        assert np.array_equal(a, b), (k, float(np.max(np.abs(a - b))))


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("count", [1, 3, 4, 5, 63])
def test_samples_do_not_depend_on_their_number(precision, count):
    """Four samples per workgroup: the first `count` rows of 64 samples, to the
    bit, and nothing past them."""
    torch = pytest.importorskip("torch")
    s = pa.Solver.from_problem(_state_problem(7, (19, 23), (P, X), 61, precision=precision))
    s.advance(4)
    pts = np.random.default_rng(7).integers(0, 19, (64, 2)).astype(np.int32)
    out = []
    for n in (64, count):
        feat = torch.full((64, 128), -7.0, device="cuda")
        targ = torch.full((64, 6), -7.0, device="cuda")
        s.closure_samples(pts[:n], feat, targ)
        out.append((feat.cpu().numpy(), targ.cpu().numpy()))
    for all_, some in zip(*out):
        assert np.array_equal(some[:count], all_[:count]) and np.all(some[count:] == -7.0)
        assert np.isfinite(all_).all() and np.any(all_ != 0)
    s.close()
