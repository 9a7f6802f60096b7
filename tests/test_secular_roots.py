"""The root finder of the divide and conquer, from the header that the kernels include, compiled for the CPU: where its iteration may end."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("secular") / "driver")
    b = subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I" + os.path.join(ROOT, "paper_2207_04228_amd", "csrc"),
                        os.path.join(ROOT, "tests", "secular_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-4000:]
    return exe


@pytest.mark.parametrize("spread", [1.0, 1e-4])
@pytest.mark.parametrize("poles, merges", [(4, 12000), (8, 12000), (16, 8000), (64, 1000), (128, 400)])
def test_last_root_of_a_merge(driver, poles, merges, spread):
    """Right of all poles the interpolation is of second order.  The iteration ends at a residual of 4 units of rounding of the sums (one more from the
    rounding of the sums themselves), or before a step that leaves no more than that."""
    r = subprocess.run([driver, str(poles), str(merges), str(spread)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    print(r.stdout.strip())
    last, inner, most, left = (float(x) for x in r.stdout.split())
    assert last <= 5.0
    assert most <= 8 and left == 0
