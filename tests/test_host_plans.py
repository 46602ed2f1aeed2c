"""The work splits of the products and the row sums on the CPU, under the address
and undefined-behaviour sanitizers: the extents of their partial sums over the
whole range of sizes, and the fixed-point column sums of a single column."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host", "plan_check.cpp")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("hostplans") / "plan_check")
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-Wall", "-Wextra", "-Werror",
           "-I", os.path.join(ROOT, "paper_2609_38198_amd", "csrc"), SRC, "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return out


@pytest.mark.parametrize("mode", ["prefixes", "products"])
def test_extents_of_partial_sums(driver, mode):
    res = subprocess.run([driver, mode], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr


def test_single_column_sums(driver):
    res = subprocess.run([driver, "columns"], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
