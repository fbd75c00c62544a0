"""The library's planning rules (rr_plan.h) on the CPU, over all the values
that its entry points accept."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GXX = shutil.which("g++")
pytestmark = pytest.mark.skipif(GXX is None, reason="no host compiler")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    subprocess.run([GXX, "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "paper_2502_13245_amd", "csrc"),
                    os.path.join(ROOT, "tests", "plan", "plan_driver.cpp"), "-o", exe], check=True)

    def run(*args):
        p = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)
        return p.returncode, p.stdout
    return run


def test_beam_scratch_and_lds(driver):
    rc, out = driver("lds")
    assert rc == 0, out


def test_task_list_stays_in_its_capacity(driver):
    rc, out = driver("list")
    assert rc == 0, out
    # a margin that leaves out the seeds already drawn is told apart
    rc, out = driver("list-drawn")
    assert rc == 1 and "points in a list" in out


def test_dense_scans_load_the_xcds_evenly(driver):
    rc, out = driver("scan")
    assert rc == 0, out
