"""The alignment gradient of a batch anywhere in the hit arrays: the indices the
reduction loads (in a host build), and a batch of empty tracks at the arrays'
end, which contributes nothing."""
import os
import subprocess

import numpy as np
import pytest
import torch

from toygen import generate, workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_loads_stay_within_the_arrays(tmp_path):
    exe = str(tmp_path / "align")
    src = os.path.join(ROOT, "tests", "hostcheck", "kf_align_check.cpp")
    subprocess.run(["hipcc", "--offload-host-only", "-x", "hip", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2312_11728_amd", "csrc"), "-o", exe, src], check=True,
                   capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
def test_empty_tracks_at_the_end(dt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("empty tracks at the arrays' end", dt, flush=True)
    n, dev = 70, torch.device("cuda", 0)
    ev = generate(workloads()["barrel10"], n)
    t = K.event_tensors(ev, dt, dev)
    geom = K.Geometry.from_toy(ev.geometry)
    off = torch.full((n + 1,), ev.n_hits, dtype=torch.int32, device=dev)
    hits = (off, t["hit_layer"], t["hit_valid"], t["hit_pos"], t["hit_cov"])
    ctx = K.Context(0)
    try:
        st, cov, q, _ = ctx.make_seeds(t["hit_offsets"], t["hit_valid"], t["hit_pos"], ev.geometry.bz)
        ck = torch.zeros(28, n * 9, dtype=dt, device=dev)
        out = ctx.fit_tracks(st, cov, q, *hits, geom, checkpoints=ck, seg=1, max_len=10)
        gs, _, ga = ctx.fit_adjoint(st, cov, q, *hits, geom, ck, 1, 10, out["status"])
        torch.cuda.synchronize()
        assert not np.any(ga.cpu().numpy()) and not np.any(gs.cpu().numpy())
    finally:
        ctx.close()
