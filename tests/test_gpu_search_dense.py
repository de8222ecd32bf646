"""A window with more hits than a slot's scan puts aside (24, read 8 at a
time): copies of every hit, a hair's breadth apart and with ids that rank them,
crowd every window with accepted hits, so that the lists fill and are scored
several times per window; the lists equal the oracle's."""
import numpy as np
import pytest
import torch

from oracle import kf_search as KS
from search_common import PLAN, SEED_LAYER, default_params, f32, search_inputs
from test_gpu_search import compare, gpu_search

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies,beam", [(7, 6), (8, 2), (25, 4), (60, 6)])
def test_crowded_windows(copies, beam):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("crowded windows", copies, beam, flush=True)
    _, _, g, pools, p, C, q = search_inputs(40, noise=False)
    plan = PLAN[:5]
    rng = np.random.default_rng(copies)
    rep = lambda a: np.repeat(a, copies, axis=-1)
    pools.pos = rep(pools.pos)
    pools.pos[2] = f32(pools.pos[2] + rng.uniform(-0.02, 0.02, pools.pos.shape[1]))
    pools.cov = rep(pools.cov)
    pools.hit_id = rng.permutation(pools.pos.shape[1]).astype(pools.hit_id.dtype)
    pools.layer_offsets = np.asarray(pools.layer_offsets) * copies
    if getattr(pools, "module", None) is not None:
        pools.module = rep(pools.module)
    o = KS.score_hits(p, C, q, np.full(40, SEED_LAYER), plan, g, pools, default_params(g, beam))
    ctx = K.Context(0)
    try:
        gs = gpu_search(ctx, K, g, pools, p, C, q, plan=plan, beam=beam)
    finally:
        ctx.close()
    # near ties between a hit's copies flag seeds; the others agree exactly,
    # and (with the default beam) a flagged seed's result is one that the
    # search can give
    compare(gs, o, max_flag_frac=1.0, inputs=(p, C, q, g, pools, plan) if beam == 6 else None)
