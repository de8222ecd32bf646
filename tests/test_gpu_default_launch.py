"""A fit whose caller chose no launch shape runs the staged kernel in FP32 and the
direct one in FP64, in blocks by size, with the same bits either way: those of
the direct layout chosen explicitly, at the sizes where the block changes, with
and without checkpoints."""
import pytest
import torch

from toygen import generate, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("name,n", [("barrel20", 1), ("mixed26", 63), ("mixed26", 4099), ("barrel20", 16384),
                                    ("barrel20", 16385), ("barrel20", 35001), ("mixed26", 56001)])
def test_default_launch_has_the_direct_layouts_bits(name, n, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("default launch", name, n, dtype, flush=True)
    dev = torch.device("cuda", 0)
    ev = generate(workloads()[name], n)
    t = K.event_tensors(ev, dtype, dev)
    hits = (t["hit_offsets"], t["hit_layer"], t["hit_valid"], t["hit_pos"], t["hit_cov"])
    geom = K.Geometry.from_toy(ev.geometry)
    max_len, seg = 26, 5
    out = []
    for chosen in (False, True):
        c = K.Context(0)
        try:
            if chosen:
                c.set_fit_launch(dtype, 256, 0, 4, 1, 0)
            ck = torch.zeros(28, n * K.n_checkpoint_segments(max_len, seg), dtype=dtype, device=dev)
            f = c.seed_fit_tracks(*hits, geom, 1, max_len=max_len)
            h = c.seed_fit_tracks(*hits, geom, 1, checkpoints=ck, seg=seg, max_len=max_len)
            torch.cuda.synchronize()
            keep = ("state", "cov", "charge", "chi2", "ndf", "status")
            out.append([x[k].cpu() for x in (f, h) for k in keep] + [ck.cpu()])
        finally:
            c.close()
    for x, y in zip(*out):
        assert torch.equal(x, y) or torch.equal(x.nan_to_num(7.0), y.nan_to_num(7.0))
