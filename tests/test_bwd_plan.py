"""The split backward core's plan on the CPU: where its waves meet and which ring
cells they read, for every small case (tests/bwd_plan_check.cpp, compiled with the header that the kernel
uses)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "bwd_plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2501_07331_amd", "csrc"),
                    "-o", exe, os.path.join(ROOT, "tests", "bwd_plan_check.cpp")], check=True)
    return lambda *a: subprocess.run([exe, *a], capture_output=True, text=True, timeout=100)


def test_no_wave_overtakes_another_one_that_reads_the_ring(check):
    r = check()
    assert r.returncode == 0, r.stdout


def test_terms_read_their_arrival_or_a_complete_row(check):
    assert check().stdout.splitlines()[0] == "0 wrong cells"


def test_the_check_finds_a_missing_meeting(check):
    """Without the barrier before the steps past the last spikes, a wave may
    write the row of those spikes again while another one reads it."""
    r = check("no-tail")
    assert r.returncode == 1 and ", 0 with a race" not in r.stdout, r.stdout
