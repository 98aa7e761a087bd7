"""The host's plans (csrc/ob_plan.h) without a device: order of the workgroups that wait for others, numbering of the
arrivals at the layers' barriers, and the rules that say which kernel a list takes.  Over random tensor lists, in a
program of its own with checked containers."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_tables")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-D_GLIBCXX_ASSERTIONS", "-fsanitize=undefined",
                    "-fno-sanitize-recover=undefined", "-I", os.path.join(ROOT, "paper_2104_06069_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "plan_tables.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("check", ["trail", "ratios_trail", "big_rule", "arrivals", "second_reads", "small_lists"])
def test_plan(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.stdout, r.stderr[-2000:])
