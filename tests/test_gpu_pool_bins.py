"""The ways the hit pool is binned: by buckets of bins (a bucket's hits in one
go or, beyond what LDS holds, in two passes; buckets of 2^10 to 2^13 bins) or
hit by hit (pools above 2^25 hits, binnings above 2^25 bins).  Hits that no
window reaches are added to a pool so that each way is taken, and the search
must give the same lists, scores and status bits as on the pool alone: the
ranking is a total order, so nothing depends on the order within a bin."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from search_common import search_inputs
from test_gpu_search import gpu_search

pytestmark = pytest.mark.gpu


def with_decoys(pools, layer, pos, dev):
    """The pool on the device with hits at pos [3, k] added to a layer."""
    k = pos.shape[1]
    f = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), device=dev).to(dt)
    at = int(pools.layer_offsets[layer + 1])
    off = np.array(pools.layer_offsets).copy()
    off[layer + 1:] += k
    put = lambda a, b: torch.cat((a[..., :at], b, a[..., at:]), dim=-1).contiguous()
    cov = torch.zeros(6, k, device=dev)
    cov[0] = cov[2] = cov[5] = 1e-4
    dev_pool = (put(f(pools.pos, torch.float32), pos), put(f(pools.cov, torch.float32), cov),
                put(f(pools.hit_id, torch.int32), torch.arange(k, dtype=torch.int32, device=dev) + 10**8))
    return SimpleNamespace(layer_offsets=off), dev_pool


# layer 10 is searched, layer 0 is not
@pytest.mark.parametrize("layer,n,half_z,spot", [
    (10, 1, 150.0, True),            # buckets of 2^10 bins
    (10, 5000, 150.0, True),         # one of them in two passes
    (0, 3000, 150000.0, False),      # 17.8M bins: buckets of 2^13
    (0, 3000, 400000.0, False),      # 43M bins: hit by hit
    (0, (1 << 25) + 5, 150.0, False),   # pool above 2^25 hits: hit by hit
])
def test_every_way_of_binning_gives_the_same_search(layer, n, half_z, spot):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("pool binning", layer, n, half_z, flush=True)
    _, _, g, pools, p, C, q = search_inputs(150)
    dev = torch.device("cuda", 0)
    ctx = K.Context(0)
    try:
        ref = gpu_search(ctx, K, g, pools, p, C, q)
        gen = torch.Generator(device=dev).manual_seed(7)
        u = torch.rand(2, n, generator=gen, device=dev)
        phi = 0.3 + 0.02 * u[0] if spot else (2.0 * u[0] - 1.0) * np.pi
        z = 140.0 + 0.5 * u[1] if spot else (2.0 * u[1] - 1.0) * half_z
        R = float(g.pos[layer])
        more, dev_pool = with_decoys(pools, layer, torch.stack((R * torch.cos(phi), R * torch.sin(phi), z)), dev)
        lo, hi = np.array(g.lo, float), np.array(g.hi, float)
        lo[layer], hi[layer] = -half_z, half_z
        wide = type(g)(**{**g.__dict__, "lo": lo, "hi": hi})
        got = gpu_search(ctx, K, wide, more, p, C, q, dev_pool=dev_pool)
    finally:
        ctx.close()
    assert (ref["hits"] >= 0).any()
    for k in ("hits", "score", "status", "state"):
        assert np.array_equal(ref[k], got[k], equal_nan=True), k
