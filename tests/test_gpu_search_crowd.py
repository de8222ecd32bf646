"""Windows with many times the hits that a slot's scan puts aside (24, read 8 at
a time), whose ranking the oracle decides: copies of every hit spread over the
window, so that their chi2 differ by far more than FP32 rounding.  A hit lost or
scored twice where a full list is scored in the middle of a window would change
the lists or the scores."""
import numpy as np
import pytest
import torch

from oracle import kf_search as KS
from search_common import PLAN, SEED_LAYER, default_params, f32, search_inputs
from test_gpu_search import compare, gpu_search

pytestmark = pytest.mark.gpu
N = 60


@pytest.mark.parametrize("copies,arc,beam,layers", [(120, 0.02, 2, 4), (120, 0.02, 4, 2), (300, 0.03, 2, 2),
                                                    (120, 0.025, 6, 2), (200, 0.02, 1, 5)])
def test_crowded_windows_ranked(copies, arc, beam, layers):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("ranked crowd", copies, beam, layers, flush=True)
    g, pools, p, C, q, plan = crowd(copies, arc, layers)
    prm = default_params(g, beam)
    o = KS.score_hits(p, C, q, np.full(N, SEED_LAYER), plan, g, pools, prm)
    # the windows hold more than the list on average, and nearly all seeds are decided
    assert o["n_window_hits"] > 1.3 * 24 * N * (1 + beam * (layers - 1))
    assert o["flagged"].mean() <= 0.2
    ctx = K.Context(0)
    try:
        gs = gpu_search(ctx, K, g, pools, p, C, q, plan=plan, beam=beam)
    finally:
        ctx.close()
    same = compare(gs, o)
    for s in np.nonzero(~same)[0]:   # flagged: a result that the search can give
        ok, _ = KS.valid_alternative(gs["hits"][s], p[s], C[s], q[s], SEED_LAYER, plan, g, pools, prm, budget=16)
        if not ok:
            ok, why = KS.consistent_result(gs["hits"][s], gs["score"][s], p[s], C[s], q[s], SEED_LAYER, plan, g, pools,
                                           prm, o["hits"][s], o["score"][s], o["score_err"][s])
            assert ok, (s, why)


def crowd(copies, arc, layers):
    """N seeds; every hit `copies` times, moved by up to 0.3 cm along z and
    `arc` cm along r-phi."""
    _, _, g, pools, p, C, q = search_inputs(N, noise=False)
    rng = np.random.default_rng(1)
    n = pools.pos.shape[1]
    dz, da = rng.uniform(-0.3, 0.3, (n, copies)), rng.uniform(-arc, arc, (n, copies))
    dz[:, 0] = da[:, 0] = 0.0
    x, y, z = np.repeat(pools.pos, copies, axis=-1)
    r, phi = np.hypot(x, y), np.arctan2(y, x) + da.reshape(-1) / np.hypot(x, y)
    pools.pos = f32(np.stack([r * np.cos(phi), r * np.sin(phi), z + dz.reshape(-1)]))
    pools.cov = np.repeat(pools.cov, copies, axis=-1)
    pools.hit_id = rng.permutation(n * copies).astype(pools.hit_id.dtype)
    pools.layer_offsets = np.asarray(pools.layer_offsets) * copies
    return g, pools, p, C, q, PLAN[:layers]
