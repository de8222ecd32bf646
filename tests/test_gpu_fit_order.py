"""The staged fit with its tracks sorted by length within groups of 2048, the
groups dealt out to the chip's eight dies in sets of eight: batches that end
inside a group, at a set's edge and beyond, for every block size, give the
bits of the staged fit in track order."""
import numpy as np
import pytest
import torch

from toygen import generate, truncate, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 65, 2048, 2049, 8 * 2048, 8 * 2048 + 1, 17 * 2048 - 3])
def test_sorted_and_track_order_agree(n, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("sorted fit", n, dtype, flush=True)
    dev = torch.device("cuda", 0)
    ev = generate(workloads()["mixed26"], n)
    ev = truncate(ev, (np.arange(n) + 5) % 27)   # also tracks without entries
    t = K.event_tensors(ev, dtype, dev)
    hits = (t["hit_offsets"], t["hit_layer"], t["hit_valid"], t["hit_pos"], t["hit_cov"])
    geom = K.Geometry.from_toy(ev.geometry)
    c = K.Context(0)
    try:
        c.reserve(n, 26)
        out = []
        for layout, block, persistent in ((3, 256, 0), (4, 256, 0), (4, 64, 0), (4, 192, 0), (4, 256, 1)):
            c.set_fit_launch(dtype, block, persistent, 1, 1, layout)
            f = c.seed_fit_tracks(*hits, geom, 1, max_len=26)
            torch.cuda.synchronize()
            out.append({k: f[k].cpu() for k in ("state", "cov", "charge", "chi2", "ndf", "status")})
    finally:
        c.close()
    for o in out[1:]:
        for k in o:
            assert torch.equal(out[0][k].nan_to_num(7.0) if o[k].is_floating_point() else out[0][k],
                               o[k].nan_to_num(7.0) if o[k].is_floating_point() else o[k]), k
