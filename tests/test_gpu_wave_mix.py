"""A track's results do not depend on the tracks beside it: the same tracks
mixed in one wave (barrel and disk crossings side by side, which a wave takes
by the general transport) and alone in waves of their own (64 copies each: a
wave between barrel layers takes the shorter form) give the same bits."""
import numpy as np
import pytest
import torch

from toygen import generate, workloads

pytestmark = pytest.mark.gpu
N = 48


@pytest.fixture(scope="module")
def kf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as _kf
    return _kf


def _tracks(K, dtype):
    """N tracks of mixed26, half of them central, as tensors; and the same
    tracks 64 times each."""
    ev = generate(workloads()["mixed26"], 4000)
    kind = np.asarray(ev.geometry.kind)
    off = np.asarray(ev.hit_offsets)
    barrel = np.array([(kind[ev.hit_layer[off[t]:off[t + 1]]] == 0).all() for t in range(4000)])
    pick = np.stack([np.flatnonzero(barrel & (ev.lengths() >= 8))[:N // 2],
                     np.flatnonzero(~barrel & (ev.lengths() >= 8))[:N // 2]], 1).reshape(-1)
    t = K.event_tensors(ev, dtype, torch.device("cuda", 0))

    def batch(tracks):
        length = off[tracks + 1] - off[tracks]
        new = np.concatenate([[0], np.cumsum(length)])
        idx = torch.from_numpy(np.repeat(off[tracks] - new[:-1], length) + np.arange(new[-1])).to(t["hit_pos"].device)
        return (torch.from_numpy(new.astype(np.int32)).to(idx.device), t["hit_layer"][idx].contiguous(),
                t["hit_valid"][idx].contiguous(), t["hit_pos"][:, idx].contiguous(), t["hit_cov"][:, idx].contiguous())

    return ev, batch(pick), batch(np.repeat(pick, 64))


def _equal(a, b):
    """b holds every column of a 64 times."""
    a = a.reshape(-1, a.shape[-1])
    b = b.reshape(a.shape[0], a.shape[1], 64)
    return bool((torch.nan_to_num(a, 7.0)[:, :, None] == torch.nan_to_num(b, 7.0)).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_propagate(kf, dtype):
    print("propagate in mixed waves", dtype, flush=True)
    ev, one, _ = _tracks(kf, dtype)
    geom = kf.Geometry.from_toy(ev.geometry)
    ctx = kf.Context(0)
    try:
        p, c, q, _ = ctx.make_seeds(one[0], one[2], one[3], ev.geometry.bz, 1)
        first = one[0][:-1].long()
        target = one[1][first + 5].contiguous()   # the sixth hit's layer
        many = lambda x: x.repeat_interleave(64, -1).contiguous()
        a = ctx.propagate(p, c, q, target, geom)
        b = ctx.propagate(many(p), many(c), many(q), many(target), geom)
        torch.cuda.synchronize()
        kinds = np.asarray(ev.geometry.kind)[target.cpu().numpy()]
        assert set(kinds) == {0, 1}
        for x, y in zip(a, b):
            if torch.is_tensor(x):
                assert _equal(x, y)
    finally:
        ctx.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("seg,no_alloc", [(1, False), (5, False), (5, True)])
def test_fit_and_gradient(kf, dtype, seg, no_alloc):
    print("gradient in mixed waves", dtype, seg, no_alloc, flush=True)
    ev, one, many = _tracks(kf, dtype)
    geom = kf.Geometry.from_toy(ev.geometry)
    ctx = kf.Context(0)
    got = []
    try:
        for hits in (one, many):
            n = hits[0].numel() - 1
            p, c, q, _ = ctx.make_seeds(hits[0], hits[2], hits[3], ev.geometry.bz, 1)
            ck = torch.zeros(28, n * kf.n_checkpoint_segments(26, seg), dtype=dtype, device=p.device)
            f = ctx.fit_tracks(p, c, q, *hits, geom, checkpoints=ck, seg=seg, max_len=26)
            gs, gh, _ = ctx.fit_adjoint(p, c, q, *hits, geom, ck, seg, 26, f["status"], no_alloc=no_alloc)
            torch.cuda.synchronize()
            got.append((f, gs, gh))
    finally:
        ctx.close()
    (f, gs, gh), (fm, gsm, ghm) = got
    for k in ("state", "cov", "chi2"):
        assert _equal(f[k], fm[k]), k
    assert _equal(gs, gsm)
    o, om = one[0].cpu().numpy(), many[0].cpu().numpy()
    for t in range(N):
        for copy in (0, 63):
            a = om[64 * t + copy]
            assert torch.equal(gh[:, o[t]:o[t + 1]].nan_to_num(7.0), ghm[:, a:a + o[t + 1] - o[t]].nan_to_num(7.0)), t
