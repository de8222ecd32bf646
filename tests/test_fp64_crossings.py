"""The two FP64 crossings of the device code against each other, in a host build."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("contract", ["off", "fast"])
def test_crossings_agree(tmp_path, contract):
    exe = str(tmp_path / "crossings")
    subprocess.run(["hipcc", "--offload-host-only", "-x", "hip", "-O2", "-std=c++17", "-ffp-contract=" + contract,
                    "-mfma", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2312_11728_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "hostcheck", "kf_crossing_check.cpp")],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
