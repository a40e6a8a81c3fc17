"""Host checks of the sub-grids in LDS: their kernel against the staged
plans', and the rule that takes a batch's series there
(tests/subgrid_check.cpp, no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2409_08090_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = tmp_path_factory.mktemp("subgrid") / "subgrid_check"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I/opt/rocm/include", "-D__HIP_PLATFORM_AMD__",
                    os.path.join(HERE, "subgrid_check.cpp"), os.path.join(CSRC, "plan.cpp"),
                    os.path.join(CSRC, "chip_tables.cpp"), "-o", str(exe)], check=True)

    def run(what):
        r = subprocess.run([str(exe), what], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
        assert r.stdout.strip().endswith("ok")

    return run


def test_as_accurate_as_the_staged_plan_of_the_series(check):
    check("accuracy")


def test_batches_take_the_path_that_was_timed_shorter(check):
    check("choice")


def test_single_calls_take_the_path_that_was_timed_shorter(check):
    check("single")


def test_every_choice_fits_the_kernels(check):
    check("forms")


def test_first_call_at_a_tolerance_is_not_held_up_by_its_tables(check):
    check("time")


def test_tables_lie_where_their_layout_says(check):
    check("tables")
