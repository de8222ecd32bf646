"""The reverse sweep of tracks that the forward fit stopped, or whose crossing is
on the edge of existing, in a host build of the device code."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stop") / "stop")
    subprocess.run(["hipcc", "--offload-host-only", "-x", "hip", "-O1", "-g", "-std=c++17",
                    "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=all", "-Wno-unused-command-line-argument",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2312_11728_amd", "csrc"),
                    "-o", out, os.path.join(ROOT, "tests", "hostcheck", "kf_stop_check.cpp")],
                   check=True, capture_output=True, timeout=300)
    return out


@pytest.mark.parametrize("check", ["step", "done", "layer"])
def test_stops(exe, check):
    r = subprocess.run([exe, check], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]
