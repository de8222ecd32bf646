"""A track's final fit does not depend on the batch it is in: every round
gathers the tracks still open in blocks of 128, in whatever order the blocks
finish, and judges the hits 16 or 4 entries at a time by the batch's size.
Tracks of a large batch and of small ones cut from it (ends inside and at the
edges of the blocks; a low cut, so that most tracks stay open for several
rounds; mixed lengths with holes) give the same bits."""
import numpy as np
import pytest
import torch

from test_gpu_final import ctx, gpu_final, kf, planted  # noqa: F401  (fixtures)
from toygen import generate, subset, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("name,n,mode", [("barrel20", 13200, 0), ("mixed26", 10300, 1)])
def test_small_batches_cut_from_a_large_one(ctx, kf, name, n, mode, dtype):  # noqa: F811
    print("final fit, batch split", name, n, dtype, flush=True)
    ev = planted(generate(workloads()[name], n), every=3)
    kw = dict(seed_mode=mode, chi2_cut=6.0, max_reject=3)
    whole = gpu_final(ctx, kf, ev, dtype, **kw)
    lost = np.add.reduceat(whole["outlier"].astype(np.int64), ev.hit_offsets[:-1])
    assert set(lost) == {0, 1, 2, 3}   # tracks closed in every round
    again = gpu_final(ctx, kf, ev, dtype, **kw)
    for k in whole:
        assert np.array_equal(whole[k], again[k], equal_nan=True), k
    for lo, hi in ((0, 1), (1, 128), (128, 256), (256, 385), (385, 1030), (n - 2000, n)):
        part = gpu_final(ctx, kf, subset(ev, np.arange(lo, hi)), dtype, **kw)
        e0, e1 = ev.hit_offsets[lo], ev.hit_offsets[hi]
        for k in whole:
            ref = whole[k][e0:e1] if k in ("outlier", "hit_chi2") else whole[k][lo:hi]
            assert np.array_equal(ref, part[k], equal_nan=True), (k, lo, hi)
