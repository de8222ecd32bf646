"""The shortcut of the barrel crossing against the full rule, bit for bit, in a
host build of the device code."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("contract", ["off", "fast"])
def test_near_root_is_the_full_rule(tmp_path, contract):
    exe = str(tmp_path / "roots")
    src = os.path.join(ROOT, "tests", "hostcheck", "kf_root_check.cpp")
    inc = os.path.join(ROOT, "paper_2312_11728_amd", "csrc")
    subprocess.run(["hipcc", "--offload-host-only", "-x", "hip", "-O2", "-std=c++17", "-ffp-contract=" + contract, "-mfma",
                    "-I", inc, "-o", exe, src], check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
