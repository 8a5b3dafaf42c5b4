"""The numbering of a register-window sweep's workgroups, enumerated on the host
from the header that the kernel and the launch code share: every tile of every m
range once, and no tile outside the grid."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1211_2205_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("order") / "window_order")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fsanitize=undefined",
                           "-fno-sanitize-recover=all", "-I", CSRC, "-o", exe,
                           os.path.join(HERE, "window_order_driver.cpp")])
    return exe


def test_no_group_is_empty_or_missing(driver):
    r = subprocess.run([driver, "groups", "1000000"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


def test_rows_of_the_tallest_grids(driver):
    r = subprocess.run([driver, "rows"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("strip", [0, 1, 8, -8, 5, -3, 1000])
@pytest.mark.parametrize("ntx,nty", [(1, 1), (3, 1), (7, 9), (8, 64), (1, 767), (24, 32), (769, 1), (31, 33),
                                     (23, 1471), (24, 1473), (33793, 1), (1, 33793), (42, 1301)])
def test_every_tile_of_every_range_once(driver, ntx, nty, strip):
    r = subprocess.run([driver, "tiles", str(ntx), str(nty), str(strip)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    got = np.array(r.stdout.split(), dtype=np.int64).reshape(-1, 3)
    assert got.min() >= 0 and (got.max(axis=0) < (2, ntx, nty)).all()
    flat = (got[:, 0] * nty + got[:, 2]) * ntx + got[:, 1]
    assert np.array_equal(np.sort(flat), np.arange(2 * ntx * nty))
