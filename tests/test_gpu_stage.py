"""The staged fits read their hits through 32-bit byte offsets while every hit
array is below 4 GB and through 64-bit ones beyond: the same tracks at the end
of larger arrays, seeds and both directions, give the same bits."""
import numpy as np
import pytest
import torch

from toygen import generate, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,past", [(torch.float32, 1 << 30), (torch.float64, 1 << 29)])
def test_hits_beyond_4_gb(dtype, past):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("hits beyond 4 GB", dtype, flush=True)
    dev = torch.device("cuda", 0)
    ev = generate(workloads()["mixed26"], 321)
    t = K.event_tensors(ev, dtype, dev)
    geom = K.Geometry.from_toy(ev.geometry)
    nh = ev.n_hits
    big = past + nh
    lay = torch.empty(big, dtype=torch.int16, device=dev)
    val = torch.empty(big, dtype=torch.uint8, device=dev)
    pos = torch.empty(3, big, dtype=dtype, device=dev)
    cov = torch.empty(6, big, dtype=dtype, device=dev)
    for a, k in ((lay, "hit_layer"), (val, "hit_valid"), (pos, "hit_pos"), (cov, "hit_cov")):
        a[..., past:] = t[k]
    lay[0], val[0] = 0, 0     # what the slots without a track read
    pos[:, 0], cov[:, 0] = 1.0, 1.0
    c = K.Context(0)
    try:
        c.set_fit_launch(dtype, 64, 0, 1, 1, 3)
        out = []
        for hits in ((t["hit_offsets"], t["hit_layer"], t["hit_valid"], t["hit_pos"], t["hit_cov"]),
                     (t["hit_offsets"] + past, lay, val, pos, cov)):
            f = c.seed_fit_tracks(*hits, geom, 1)
            b = c.backward_fit(f, *hits, geom)
            out.append({k + str(i): x[k].clone() for i, x in enumerate((f, b)) for k in x})
        torch.cuda.synchronize()
        for k in out[0]:
            assert torch.equal(out[0][k].nan_to_num(7.0), out[1][k].nan_to_num(7.0)), k
    finally:
        c.close()
