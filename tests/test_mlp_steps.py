"""The trainer's step count over steps that fail: an update that was never
launched does not count in Adam's bias correction (1 - beta1^t)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("mlp") / "mlp_steps")
    csrc = os.path.join(ROOT, "paper_1211_2205_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__=1", "-w", "-ffunction-sections",
                           "-Wl,--gc-sections", "-I", os.path.join(ROCM, "include"), "-I", csrc, "-o", exe,
                           os.path.join(HERE, "mlp_steps_driver.cpp"), os.path.join(csrc, "closure.cpp")])
    return exe


@pytest.mark.parametrize("fails", [[0, 0, 0], [0, 1, 0, 0], [2, 0, 0], [0, 3, 3, 0], [1, 2, 3, 0]])
def test_failed_steps_do_not_count(driver, fails):
    out = subprocess.run([driver] + [str(f) for f in fails], capture_output=True, text=True, check=True).stdout
    rows = [(int(a), float(b)) for a, b in (ln.split() for ln in out.splitlines())]
    done = 0
    for f, (rc, c1) in zip(fails, rows):
        assert (rc != 0) == (f != 0)
        if f == 0:
            done += 1
            assert c1 == pytest.approx(1.0 - 0.9 ** done, rel=1e-6)  # a float of it
    assert len(rows) == len(fails)
