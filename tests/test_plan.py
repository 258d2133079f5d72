"""What the host decides before a launch (bz_plan.hpp), on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_29942_amd", "csrc")


def test_plans(tmp_path):
    exe = os.path.join(str(tmp_path), "plan_checks")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-DBZ_HD=inline", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "plan_checks.cpp"), "-o", exe],
                   check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert all(line.startswith("OK ") for line in out.stdout.splitlines()) and out.stdout
