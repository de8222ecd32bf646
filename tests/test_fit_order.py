"""The order of the length-sorted staged fit, in a host build."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_order_is_a_permutation(tmp_path):
    exe = str(tmp_path / "order")
    subprocess.run(["hipcc", "--offload-host-only", "-x", "hip", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "paper_2312_11728_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "hostcheck", "kf_order_check.cpp")],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
