"""The diff kernel's grid for a unit count, a group and a limit (host code)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_diff_grid(tmp_path):
    exe = str(tmp_path / "diff_grid")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror",
                        "-I" + os.path.join(ROOT, "paper_1808_00117_amd", "csrc"),
                        os.path.join(ROOT, "tests", "c", "diff_grid_test.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "diff grid: ok" in r.stdout, r.stdout + r.stderr
