"""The library's host code without a device: each test runs a small program in a
process whose HIP calls go to tests/fake_hip.cpp (memory from the heap, launches
that do nothing), and looks at the choices the library makes."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PREAMBLE = """
import ctypes, os, sys
fake = ctypes.CDLL({fake!r}, ctypes.RTLD_GLOBAL)
sys.path.insert(0, {root!r})
import paper_1211_2205_amd as pa
import workloads as wl

def problem(N=7, n=(40, 24), precision="fp64", general=False):
    one = lambda t, x, y: 1.0 + 0.0 * x
    return wl.Problem(name="host", N=N, n=n, ax=(0.0, 1.0, 0.0, 1.0), bc=("periodic", "extrapolation"), cfl=0.5,
                      t_final=0.1, precision=precision, sigma_a=one, sigma_s0=one,
                      sigma_sl=(lambda l, t, x, y: 0.5 ** l + 0.0 * x) if general else None,
                      source={{k: one for k in range(pa.num_moments(N) if general else 1)}})

def solver(*a, **k):
    s = pa.Solver.from_problem(problem(*a, **k))
    s.advance(1)
    return s

def tile(s):
    return s.variant()[0], s.chunk_width()
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    fake = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-I",
                           os.path.join(rocm, "include"), "-o", fake, os.path.join(HERE, "fake_hip.cpp")])

    def run(body, **env):
        code = PREAMBLE.format(fake=fake, root=ROOT) + textwrap.dedent(body)
        base = {k: v for k, v in os.environ.items() if not k.startswith("STARMAP_")}
        r = subprocess.run([sys.executable, "-c", code], env={**base, **env}, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
    return run


def test_a_refused_width_is_not_a_given_one(program):
    """A width that was not taken on leaves the solver without one of its own:
    the default tile still brings its width; one that was taken on is kept."""
    program("""
        default = tile(solver())
        assert default[1] != 8
        s = pa.Solver.from_problem(problem())
        s.set_variant(0)
        s.advance(1)
        assert tile(s) == (0, 8)  # a tile given before the first device call: the widest ranges
        copies = ctypes.c_int.in_dll(fake, "fake_failing_copies")
        copies.value = 1
        try:
            s.set_chunk_width(4)
            raise SystemExit("accepted")
        except pa.StarmapError:
            pass
        assert copies.value == 0 and tile(s) == (0, 8)
        s.set_variant(-1)
        assert tile(s) == default, (tile(s), default)
        s.set_variant(0)
        s.set_chunk_width(6)
        s.set_variant(-1)
        assert tile(s) == (default[0], 6)
    """)


def test_refused_widths_leave_the_width(program):
    """With 64 KiB of LDS a 64 x 8 FP64 tile of P_13 holds four indices of m, not six."""
    program("""
        s = solver(N=13)
        s.set_chunk_width(4)
        s.set_variant(5)
        for width in (6, 8):
            try:
                s.set_chunk_width(width)
                raise SystemExit("accepted")
            except pa.StarmapError:
                assert tile(s) == (5, 4)
    """, FAKE_LDS="65536")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
def test_default_tile_after_a_batch(program, precision):
    """The tile and width that a batch gave its solvers are the batch's: the
    default tile brings its own width back, or the one the user had given."""
    program(f"""
        default = tile(solver(precision={precision!r}))
        for given in (0, 6):
            a, c = (pa.Solver.from_problem(problem(precision={precision!r})) for _ in range(2))
            if given:
                a.set_chunk_width(given)
            b = pa.Batch([a, c])
            b.run(use_graph=False)
            assert b.variant() == (0, 8) and tile(a) == tile(c) == (0, 8)
            b.close()
            a.set_variant(-1)
            c.set_variant(-1)
            assert tile(c) == default, (tile(c), default)
            assert tile(a) == (default[0], given or default[1])
    """)


@pytest.mark.parametrize("precision,storage", [("fp64", 0), ("fp32", 1), ("bf16", 2)])
def test_tune_cache_lines_name_their_tile(program, precision, storage, tmp_path):
    """A line counts if its variant number still means the tile it was written
    for: lines without a tile, from when the numbers meant other tiles, and lines
    of another tile or kernel leave the default."""
    program(f"""
        path = os.environ["STARMAP_TUNE_CACHE"]
        storage, make = {storage}, lambda: solver(precision={precision!r})

        def chosen(*rows):
            with open(path, "w") as f:
                f.writelines(r + chr(10) for r in rows)
            return tile(make())

        default = chosen()
        key = f"7 40 24 {{storage}}"
        for stale in ("4 8", "9 6", "12 4", "6 8", "0 8", "5 8 64 8", "5 6 64 8 9", "5 6 8 64 10", "5 6 64 8 -1", "5 6 64 8 x"):
            assert chosen(f"{{key}} {{stale}}") == default, stale
        # the autotuner's line is taken, over stale ones before and after it
        os.remove(path)
        s = make()
        s.autotune(1)
        tuned = tile(s)
        (line,) = open(path).read().splitlines()
        assert chosen(f"{{key}} 9 6", line, f"{{key}} 4 8", f"7 40 25 {{storage}} 1 4") == tuned
        assert chosen(line, line.replace("7 40 24", "7 41 24")) == tuned
    """, STARMAP_TUNE_CACHE=str(tmp_path / "cache"))


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
def test_closure_network_is_opted_in_on_every_device(program, precision):
    """The network's weights take more LDS than a kernel gets unasked, and what a
    kernel gets is set device by device."""
    program(f"""
        import numpy as np
        weights = np.load(os.path.join(os.path.dirname(pa.__file__), "weights", "closure_p5_256.npy"))
        device = ctypes.c_int.in_dll(fake, "fake_device")
        for device.value in (0, 1, 0, 70, 1):
            s = pa.Solver.from_problem(problem(N=5, precision={precision!r}), closure="learned")
            s.load_closure(weights)
            s.advance(1)
            t = pa.Solver.from_problem(problem(N=5, precision={precision!r}), closure="learned")
            t.load_closure(weights)
            b = pa.Batch([t])
            b.run(use_graph=False)
            b.close()
    """)


def test_default_fp64_tiles_go_by_decay_planes_and_sources(program):
    """Of grids above some 350^2 points, solvers of few orders take the LDS window
    (32 x 8 tiles, one m range) where the general sweep's look-ups or the fit of
    the tiles on the chip make it the faster one."""
    program("""
        def chosen(N, n, by_order, sources):
            p = problem(N, (n, n))
            p.bc = ("extrapolation", "extrapolation")
            one = p.sigma_a
            if by_order:
                p.sigma_sl = lambda l, t, x, y: 0.5 ** l + 0.0 * x
            if sources:
                p.source = {k: one for k in range(pa.num_moments(N))}
            s = pa.Solver.from_problem(p)
            s.advance(1)
            return tile(s)

        window, lds = lambda w: (12, w), lambda w: (8, w)
        for N, n, by_order, sources, want in (
            (4, 300, True, True, window(6)), (4, 360, False, False, window(6)), (4, 360, True, False, lds(6)),
            (4, 360, False, True, lds(6)), (4, 500, False, False, lds(6)), (4, 600, False, False, window(6)),
            (3, 360, False, False, window(4)), (3, 360, True, False, lds(4)), (3, 360, True, True, window(4)),
            (3, 500, True, True, lds(4)), (2, 360, False, False, lds(4)), (2, 440, False, False, (7, 4)), (2, 360, True, True, lds(4)), (2, 440, True, False, (7, 4)),
            (5, 360, True, False, lds(6)), (5, 360, True, True, window(6)), (5, 500, False, False, lds(6)),
            (5, 480, False, False, window(6)), (6, 360, True, False, window(4)), (6, 390, True, False, lds(8)), (6, 360, True, True, window(4)),
            (7, 360, True, False, window(4)), (1, 360, True, True, (7, 4)),
        ):
            assert chosen(N, n, by_order, sources) == want, (N, n, by_order, sources, chosen(N, n, by_order, sources))
    """)
