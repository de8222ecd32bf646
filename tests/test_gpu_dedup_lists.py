"""Duplicate removal at the edges of its lane groups (16, 32 or 64 lanes per
track) and rows (eight layers at a time), with few ids so that the lists of
shared hits are long and ids that meet in the hash table: keep and dup_of
equal the oracle's."""
import numpy as np
import pytest
import torch

from oracle import kf_dedup as D

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_layers", [1, 2, 8, 9, 16, 17, 32, 33, 64])
def test_group_edges(n_layers):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("duplicate removal", n_layers, flush=True)
    rng = np.random.default_rng(n_layers)
    n = 259
    hits = rng.integers(-2, 40, size=(n, n_layers)).astype(np.int32)
    copies = rng.integers(0, n, size=(n // 3, 2))
    hits[copies[:, 0], :(n_layers + 1) // 2] = hits[copies[:, 1], :(n_layers + 1) // 2]
    hits = np.where(hits >= 0, hits << 8, hits).astype(np.int32)
    score = rng.integers(-3, 4, size=n).astype(np.float32)   # ties
    score[::17] = -np.inf
    ctx = K.Context(0)
    try:
        for frac in (0.05, 0.5, 1.0):
            keep, dup = ctx.remove_duplicates(torch.tensor(hits, device=ctx.device),
                                              torch.tensor(score, device=ctx.device), frac)
            torch.cuda.synchronize()
            ok, od = D.remove_duplicates(hits, score, np.float32(frac))
            assert np.array_equal(keep.cpu().numpy().astype(bool), ok), frac
            assert np.array_equal(dup.cpu().numpy().astype(np.int64), od), frac
    finally:
        ctx.close()
