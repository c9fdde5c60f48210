"""The memory that a batch may take and keep for operands and stored rows is
bounded whatever is free (plan.hpp, built here with g++ for the host)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GIB = 1 << 30


@pytest.fixture(scope="module")
def budget(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and the ROCm headers")
    exe = str(tmp_path_factory.mktemp("budget") / "probe")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_1309_5478_amd", "csrc"), "-I" + os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "batch_budget_probe.cpp"), "-o", exe], check=True)

    def run(free, env=None):
        e = {k: v for k, v in os.environ.items() if k != "KNN_SPLIT_BYTES"}
        e.update(env or {})
        out = subprocess.run([exe, str(free)], env=e, capture_output=True, text=True, check=True).stdout.split()
        return tuple(int(x) for x in out)
    return run


def test_bounds(budget):
    for free in (0, 1000, GIB, 24 * GIB, 100 * GIB, 288 * GIB, 2000 * GIB):
        split, rows = budget(free)
        assert split == min(free // 3, 64 * GIB)
        assert rows == min(free // 6, 8 * GIB)


def test_caller_lowers_the_operands(budget):
    assert budget(288 * GIB, {"KNN_SPLIT_BYTES": "1000000"}) == (1000000, 8 * GIB)
    assert budget(9000, {"KNN_SPLIT_BYTES": "1000000"}) == (3000, 1500)
    assert budget(9000, {"KNN_SPLIT_BYTES": "0"}) == (3000, 1500)
