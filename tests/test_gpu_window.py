"""The register-window sweep (window.hip) at the sizes where it can go wrong:
tiles with one point of remainder, grids smaller than a tile, every remainder
of the m ranges, sources and decay planes of every order, launches of fewer
workgroups than compute units (orders split into runs) and more, a value that
is not finite.  FP64 variants run the same operations in the same order with
the window in registers or in LDS, so they must agree bit for bit."""
import os

import numpy as np
import pytest

import paper_1211_2205_amd as pa
import workloads as wl
from gpu_helpers import assert_parity, rel_l2

pytestmark = pytest.mark.gpu

P, X = wl.BC_PERIODIC, wl.BC_EXTRAPOLATION
LDS, WINDOW = 0, (4, 9, 12)  # FP64 variants
STEPS = 5

CASES = [
    # N, (nx, ny), bc, every order with its own decay and source
    (1, (2, 2), (X, X), False),
    (1, (63, 3), (P, P), True),
    (2, (64, 2), (X, P), False),
    (3, (65, 5), (P, X), True),
    (4, (127, 4), (X, X), False),
    (5, (128, 7), (X, P), True),
    (6, (129, 8), (P, P), False),
    (7, (33, 65), (X, X), True),
    (8, (257, 9), (P, X), False),
    (11, (66, 31), (X, P), False),
    (13, (191, 130), (X, X), False),
    (16, (62, 17), (P, P), True),
    (21, (31, 64), (X, X), True),
    (3, (700, 531), (X, P), False),  # several groups of 512 tiles, the last a partial one
]


def _problem(N, n, bc, general, precision="fp64"):
    rng = np.random.default_rng(17 * N + n[0])
    sa = rng.uniform(0.1, 2, size=3)
    src = {0: lambda t, x, y: np.exp(-x * x - y * y)}
    if general:
        src.update({k: (lambda k: lambda t, x, y: np.sin(k + x) * y)(k) for k in (1, 2) if N >= 1})
    return wl.Problem(
        name="window", N=N, n=n, ax=(-0.3, 0.9, 0.1, 1.3), bc=bc, cfl=0.5, t_final=0.4, precision=precision,
        sigma_a=lambda t, x, y: sa[0] + sa[1] * np.cos(2 * x) ** 2, sigma_s0=lambda t, x, y: sa[2] + 0 * x * y,
        sigma_sl=(lambda l, t, x, y: 0.8 ** l * (1 + 0 * x * y)) if general else None, source=src)


def _run(prob, init, variant, width):
    s = pa.Solver.from_problem(prob)
    for k, a in enumerate(init):
        s.set_field_array(3, k, a)
    s.bind_torch()
    s.set_variant(variant)
    s.set_chunk_width(width)
    s.advance(STEPS)
    out = s.moments()
    s.close()
    return out


def _init(prob):
    s = pa.Solver.from_problem(prob)
    s.bind_torch()
    shapes = [m.shape for m in s.moments()]
    s.close()
    return wl.random_state(5, shapes)


@pytest.mark.parametrize("N,n,bc,general", CASES)
def test_fp64_register_and_lds_windows_agree(N, n, bc, general):
    prob = _problem(N, n, bc, general)
    init = _init(prob)
    init[0][n[1] // 2, n[0] // 2] = np.inf  # spreads as inf and NaN
    for width in (4, 6, 8):
        ref = _run(prob, init, LDS, width)
        for v in WINDOW:
            got = _run(prob, init, v, width)
            for k, (a, b) in enumerate(zip(got, ref)):
                assert np.array_equal(a, b, equal_nan=True), (v, width, k)


@pytest.mark.parametrize("N,n,bc,general", CASES)
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_narrow_storage_against_fp64(precision, N, n, bc, general):
    """One tile and width against FP64, the others bit for bit against it.
    FP32: the parity bound of the suite.  BF16: every stored value is rounded
    by at most 2^-9 of itself in each of the 2 x 5 + 1 sweeps (and once at the
    start), and a sweep amplifies no error norm: 12 x 2^-9 = 0.024 of the
    norm."""
    prob = _problem(N, n, bc, general)
    init = _init(prob)
    ref = _run(prob, init, LDS, 8)
    narrow = _problem(N, n, bc, general, precision)
    one = _run(narrow, init, 0, 8)
    if precision == "fp32":
        assert_parity(one, ref, 1e-5, f"{precision} P_{N} {n}")
    else:
        assert rel_l2(one, ref) <= 0.024
    for width, variants in ((4, (1, 3, 6, 7)), (6, (2, 4, 10, 11)), (8, (5, 8, 9, 12, 13))):
        for v in variants:
            for k, (a, b) in enumerate(zip(_run(narrow, init, v, width), one)):
                assert np.array_equal(a, b), (v, width, k)


@pytest.mark.parametrize("precision,variant,width", [("fp64", 4, 4), ("fp64", 9, 6), ("fp64", 12, 8), ("fp32", 0, 8),
                                                     ("fp32", 7, 4), ("bf16", 4, 6), ("bf16", 12, 8)])
def test_batched_register_windows_equal_single_runs(precision, variant, width):
    """Instances of every m-range width and both kernels (with and without
    per-order decay planes) in one batch, as a graph replayed."""
    probs = [_problem(*c, precision) for c in CASES[:10]]
    solvers = [pa.Solver.from_problem(p) for p in probs]
    b = pa.Batch(solvers)
    b.set_variant(variant, width)
    for merged in (False, True):
        b.set_merged(merged)
        for _ in range(2):
            b.reset()
            b.run(use_graph=True)
            for p, s in zip(probs, solvers):
                t = pa.Solver.from_problem(p)
                t.bind_torch()
                t.set_variant(variant)
                t.set_chunk_width(width)
                t.run()
                for k, (x, y) in enumerate(zip(s.moments(), t.moments())):
                    assert np.array_equal(x, y), (p.N, p.n, merged, k)
                t.close()
    b.close()


def test_refused_tiles_stay_refused_after_a_register_window(monkeypatch):
    """64 x 8 FP64 tiles of P_39 do not fit the LDS at m ranges of 24: set_variant
    says so whether the variant before it was a register window or not."""
    monkeypatch.setenv("STARMAP_CHUNK_WIDTH", "24")
    prob = _problem(39, (20, 12), (X, X), False)
    for before in (LDS, 12):
        s = pa.Solver.from_problem(prob)
        s.bind_torch()
        s.set_variant(before)
        s.advance(1)
        with pytest.raises(pa.StarmapError):
            s.set_variant(5)
        s.set_chunk_width(4)
        s.set_variant(5)
        s.advance(1)
        s.synchronize()
        s.close()


@pytest.mark.parametrize("bc", [(X, X), (P, X)])
@pytest.mark.parametrize("nx", [29, 30, 31, 60, 61, 62, 63, 64, 122, 123, 124, 125, 126, 186])
def test_fp64_tiles_that_overlap_by_their_end_lanes(nx, bc):
    """Rows one point below, at and above whole pieces of 62 points: every
    point is updated once, from the neighbours the LDS window gives it."""
    prob = _problem(3, (nx, 5), bc, nx % 2 == 0)
    init = _init(prob)
    ref = _run(prob, init, LDS, 8)
    for v in WINDOW:
        for k, (a, b) in enumerate(zip(_run(prob, init, v, 4), ref)):
            assert np.array_equal(a, b), (v, k)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("N", [1, 2, 4, 9, 15, 16, 24])
def test_runs_of_orders(N, precision):
    """Launches of few waves split their orders into runs; each output still
    takes the same operations, so wider tiles of other run counts, down to one,
    give the same bits."""
    prob = _problem(N, (70, 61), (X, P), N % 2 == 0, precision)
    init = _init(prob)
    ref = _run(prob, init, 12 if precision == "fp64" else 8, 4)
    others = ((4, 4), (9, 8), (LDS, 8)) if precision == "fp64" else ((5, 4), (0, 8), (12, 6))
    for v, width in others:
        for k, (a, b) in enumerate(zip(_run(prob, init, v, width), ref)):
            assert np.array_equal(a, b), (v, width, k)


@pytest.mark.parametrize("precision,tiles", [("fp64", (LDS, 12)), ("fp32", (12, 8))])
def test_launches_of_very_many_tiles(precision, tiles):
    """2600^2 points make some 53000 tiles 64 wide and 2 high (the groups of
    tiles are rounded up, so from 33793 on they hold more than all tiles); FP32
    tiles 512 wide stay below that.  One instance by itself and in a batch."""
    prob = _problem(1, (2600, 2600), (X, X), False, precision)
    prob.t_final = 1e-4  # one step
    runs = []
    for v in tiles:
        s = pa.Solver.from_problem(prob)
        s.bind_torch()
        s.set_variant(v)
        s.run()
        runs.append(s.moments())
        s.close()
    s = pa.Solver.from_problem(prob)
    b = pa.Batch([s])
    b.set_variant(tiles[1], 4)
    b.run()
    for got in (runs[1], s.moments()):
        assert any(np.any(a) for a in got)
        for k, (x, y) in enumerate(zip(got, runs[0])):
            assert np.array_equal(x, y), k
    b.close()


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("bc", [(P, X), (P, P), (X, P)])
@pytest.mark.parametrize("nx", [191, 192, 193])
def test_row_ends_by_one_load_per_order(nx, bc, general):
    """FP32 launches of 2048 waves and more, in tiles of whole waves per row, take
    the x neighbours at row ends from one load per order: grids one point below,
    at and above whole waves, on axes that wrap and that do not, in both parities
    of the plain and the general sweep, for ranges of four, six and eight indices,
    against tiles of half a wave per row.  Single runs and batches of two."""
    shapes = {0: (64, 4), 6: (256, 2), 12: (512, 1)}
    prob = _problem(13, (nx, 350), bc, general, "fp32")
    init = _init(prob)
    ref = _run(prob, init, 2, 8)
    assert all(np.all(np.isfinite(a)) for a in ref) and all(np.any(a) for a in ref)
    for v, (tx, ty) in shapes.items():
        for width in (4, 6, 8):
            chunks = -(-14 // width)
            tiles = -(-(nx + (bc[0] == X)) // tx) * -(-(350 + (bc[1] == X)) // ty)
            assert tiles * tx * ty * chunks >= 2048 * 64
            for k, (a, b) in enumerate(zip(_run(prob, init, v, width), ref)):
                assert np.array_equal(a, b), (v, width, k)
    prob.t_final = 2e-2
    runs = []
    for v in (2, 0, 12):
        solvers = [pa.Solver.from_problem(prob) for _ in range(2)]
        for s in solvers:
            for k, a in enumerate(init):
                s.set_field_array(3, k, a)
        b = pa.Batch(solvers)
        b.set_variant(v, 6)
        b.run()
        runs.append([m for s in solvers for m in s.moments()])
        b.close()
    for got in runs[1:]:
        for k, (a, b) in enumerate(zip(got, runs[0])):
            assert np.array_equal(a, b), k


def _model(kind):
    if kind == "filtered":
        p = wl.checkerboard(N=6, n=45, t_final=0.3)
        p.filter_damping = wl.filter_damping(6, 8.0, power=4)
    elif kind == "changing media":
        p = wl.pulsed_medium(37, 4, 41)
    elif kind == "diffusion":
        p = wl.checkerboard(N=3, n=39, t_final=0.3)
        p.diffusion = lambda t, x, y: 0.002 + 0.0 * x
    else:
        p = wl.closure_instance(3, 5, 50)
    p.precision = "fp64"
    return p


@pytest.mark.parametrize("kind", ["filtered", "changing media", "diffusion", "closure", "fused closure"])
def test_models_with_either_window(kind):
    """The default FP64 tile of a model's larger grids is an LDS one, of its smaller
    ones a register window: both give the same bits, over split advances, and for
    closures (whose fused odd sweep moves the order-5 moments) in batches too."""
    weights = np.load(os.path.join(os.path.dirname(pa.__file__), "weights", "closure_p5_256.npy"))

    def solver():
        s = pa.Solver.from_problem(_model(kind), closure="learned" if "closure" in kind else "pn")
        s.bind_torch()
        if "closure" in kind:
            s.load_closure(weights)
            s.set_closure_fused(kind == "fused closure")
        return s

    runs = []
    for v, width in ((12, 4), (8, 6), (7, 4), (8, 8)):
        s = solver()
        s.set_variant(v)
        s.set_chunk_width(width)
        for k in (1, 4, 2):
            s.advance(k)
        runs.append(s.moments())
        s.close()
    assert any(np.any(a) for a in runs[0])
    for i, got in enumerate(runs[1:]):
        for k, (a, b) in enumerate(zip(got, runs[0])):
            assert np.array_equal(a, b), (i, k)
    if "closure" not in kind:
        return
    ends = []
    for v in (12, 8):
        pair = [solver(), solver()]
        b = pa.Batch(pair)
        b.set_variant(v, 6)
        b.run()
        ends.append([m for s in pair for m in s.moments()])
        b.close()
    for k, (a, b) in enumerate(zip(*ends)):
        assert np.array_equal(a, b), k
