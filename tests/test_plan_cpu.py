"""Every plan of csrc/plan.hpp, over lattices from one node to a million per
side, is one that the tile and block kernels can run (host code, no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plans_fit_the_kernels(tmp_path):
    exe = tmp_path / "plan_check"
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2501_16000_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "plan_check.cpp"), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) > 10000
