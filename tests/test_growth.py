"""CPU test of the account by which a sparse region job decides that no window can have
been lifted to its bound (growth.hpp): it may never say less than what was added, also
when small growth follows large."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("growth") / "harness")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-I",
                           os.path.join(ROOT, "paper_1503_03492_amd", "csrc"),
                           os.path.join(ROOT, "tests", "growth_harness.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("new_side", [0, 1])
@pytest.mark.parametrize("early,big,late,small", [
    (1, 1.0, 1, 1.0), (300, 1e2, 1000, 1e-3), (1000, 3.7e4, 1000, 0.9), (1, 1e8, 1023, 1.7),
    (1000, 1e-3, 1000, 1e2)])
def test_small_growth_after_large_is_not_lost(harness, early, big, late, small, new_side):
    out = subprocess.run([harness, str(early), str(big), str(late), str(small), str(new_side)],
                         capture_output=True, text=True, check=True).stdout
    part, whole = map(float, out.split())
    # 1.001 times a sum that is within 2^10 roundings of itself
    assert 1.0 <= part <= 1.0012
    assert 1.0 <= whole <= 1.0012
