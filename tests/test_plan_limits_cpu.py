"""Plans and index arithmetic at the largest sizes (host code, no GPU)."""
import os
import shutil
import subprocess

import pytest

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


def test_large_lattices_compute_few_nodes_twice(tmp_path):
    """Long flat lattices had blocks of 64 x 64 nodes for one to 36 rows."""
    assert int(run_check(tmp_path, "plan_waste_check").split()[1].strip(",")) > 1000


def test_launch_counts(tmp_path):
    assert int(run_check(tmp_path, "launch_count_check").split()[1]) > 5000


def test_served_sets(tmp_path):
    out = run_check(tmp_path, "serve_shape_check", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all")
    assert int(out.split()[1]) == 504


def test_order_of_box_sums(tmp_path):
    assert int(run_check(tmp_path, "sums_shape_check").split()[1]) == 7


def test_wrap_up_to_the_longest_side(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe, san = str(tmp_path / "wrap_check"), []
    for flag in ("-fsanitize=undefined", "-fno-sanitize-recover=all"):
        san += ["-Xarch_host", flag]
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2501_16000_amd", "csrc")]
    subprocess.run([hipcc, "-std=c++17", "-O1", "-x", "hip", "--cuda-host-only", *san, *inc, "-c",
                    os.path.join(ROOT, "tests", "host", "wrap_check.cpp"), "-o", exe + ".o"],
                   check=True)
    subprocess.run(["/opt/rocm/llvm/bin/clang++", "-fsanitize=undefined", exe + ".o", "-o", exe,
                    "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
