"""What the planner counts on: that a CU holds the block sweep's workgroups
(registers and LDS as the compiler reports them; no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from test_plan_limits_cpu import ROOT, run_check


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    csrc = os.path.join(ROOT, "paper_2501_16000_amd", "csrc")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-device-only", "-O3", "-std=c++17",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(csrc, "block.hip"),
                        "-o", str(tmp_path_factory.mktemp("block") / "block.o")],
                       capture_output=True, text=True, check=True)
    found, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"remark: .*?(Function Name|Occupancy \[waves/SIMD\]|ScratchSize \[bytes/lane\]"
                      r"|LDS Size \[bytes/block\]): (\S+)", line)
        if m and m[1] == "Function Name":
            name = m[2]
            found[name] = {}
        elif m:
            found[name][m[1].split()[0]] = int(m[2])
    return found


def test_lds_is_what_the_launch_asks_for(kernels, tmp_path):
    """LDS for eight wavefronts whatever the launch had let a CU hold 6 workgroups
    of one FP32 wavefront, where the plan counted 28."""
    assert len(kernels) > 60
    assert {k: v for k, v in kernels.items() if v["LDS"] or v["ScratchSize"]} == {}
    assert int(run_check(tmp_path, "block_fit_check").split()[1]) == 64


def test_registers_leave_the_wavefronts_that_the_plan_counts(kernels, tmp_path):
    """Periodic BGK in F16S held three wavefronts of eight rows per SIMD, not four.
    (Polynomial OReg in four rows holds six, modelled as the others' seven.)"""
    checked = 0
    for name, v in kernels.items():
        m = re.search(r"20batched_block_kernelILi(\d)ELi(\d)ELi(\d)E", name)
        coll = "0"
        if m:
            rows, eq, st = m.groups()
        else:
            m = re.search(r"12block_kernelILi(\d)ELi(\d)ELi(\d)ELi\dELi(\d)E", name)
            rows, eq, coll, st = m.groups()
        count = (3 if rows == "4" else 2) if st == "0" else (7 if rows == "4" else 4)
        polynomial = rows == "4" and st != "0" and eq == "1" and coll == "0"
        assert v["Occupancy"] >= count - polynomial, name
        checked += 1
    assert checked == len(kernels)
