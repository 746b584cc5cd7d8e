"""Plans of csrc/plan.hpp at the largest sizes (host code, no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_check(tmp_path, name, *flags):
    exe = tmp_path / name
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", *flags, "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2501_16000_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_longest_lattices(tmp_path):
    out = run_check(tmp_path, "plan_limits_check", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all")
    assert int(out.split()[1]) > 50
