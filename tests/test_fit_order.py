"""The order of the length-sorted staged fit: its places in a host build, and a
batch larger than the chip holds at once, whose groups' longest tracks run
first, against the fit in track order."""
import os
import subprocess

import numpy as np
import pytest
import torch

from toygen import generate, workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_order_is_a_permutation(tmp_path):
    exe = str(tmp_path / "order")
    subprocess.run(["hipcc", "--offload-host-only", "-x", "hip", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "paper_2312_11728_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "hostcheck", "kf_order_check.cpp")],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("groups,more", [(33, 0), (37, 5)])
def test_front_and_track_order_agree(groups, more, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("sorted fit with a front", groups, more, dtype, flush=True)
    dev, n = torch.device("cuda", 0), groups * 2048 + more
    ev = generate(workloads()["mixed26"], 2000)
    t = K.event_tensors(ev, dtype, dev)
    off = np.asarray(ev.hit_offsets)
    rng = np.random.default_rng(groups)
    pick = rng.integers(0, 2000, n)
    length = np.minimum(off[pick + 1] - off[pick], rng.integers(0, 27, n))   # also tracks without entries
    new = np.concatenate([[0], np.cumsum(length)])
    idx = torch.from_numpy(np.repeat(off[pick] - new[:-1], length) + np.arange(new[-1])).to(dev)
    hits = (torch.from_numpy(new.astype(np.int32)).to(dev), t["hit_layer"][idx].contiguous(),
            t["hit_valid"][idx].contiguous(), t["hit_pos"][:, idx].contiguous(), t["hit_cov"][:, idx].contiguous())
    geom = K.Geometry.from_toy(ev.geometry)
    ctx = K.Context(0)
    try:
        assert (n + 63) // 64 > 4 * ctx.cu_count()   # one wave per SIMD
        ctx.reserve(n, 26)
        first = None
        for layout, block, persistent in ((3, 256, 0), (4, 256, 0), (4, 64, 0), (4, 192, 0), (4, 256, 1)):
            ctx.set_fit_launch(dtype, block, persistent, 1, 1, layout)
            f = ctx.seed_fit_tracks(*hits, geom, 1, max_len=26)
            torch.cuda.synchronize()
            got = {k: f[k].clone() for k in ("state", "cov", "charge", "chi2", "ndf", "status")}
            first = first or got
            for k in got:
                a, b = (x.nan_to_num(7.0) if x.is_floating_point() else x for x in (first[k], got[k]))
                assert torch.equal(a, b), (k, layout, block, persistent)
    finally:
        ctx.close()
