"""The reverse sweep reads its hits a chunk of entries at a time (4 in FP64, 8
in FP32) from each track's last entry down.  Ragged batches with track lengths
at the chunk edges, holes and a last wave of one track: the FP64 gradients
against the oracle (per-track relative L2, 1e-6 for the hits and 1e-5 for the
seeds, 1e-8 for the alignment sum: the bounds of test_gpu_adjoint), and in
both precisions the zeros of the entries outside the fit.  seg 1 sweeps over
the checkpoints, seg 3 over the refilled states."""
import numpy as np
import pytest
import torch

from oracle import kf_oracle as O
from toygen import generate, truncate, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name,n,seg", [("align20", 65, 1), ("mixed26", 257, 1), ("mixed26", 64, 3), ("align20", 1, 1)])
def test_chunk_edges(name, n, seg, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("reverse sweep chunks", name, n, seg, dtype, flush=True)
    dev = torch.device("cuda", 0)
    ev = generate(workloads()[name], n)
    lengths = np.array([20, 17, 16, 15, 13, 12, 11, 9, 8, 7, 5, 4])[np.arange(n) % 12]
    ev = truncate(ev, lengths)
    t = K.event_tensors(ev, dtype, dev)
    hits = (t["hit_offsets"], t["hit_layer"], t["hit_valid"], t["hit_pos"], t["hit_cov"])
    geom = K.Geometry.from_toy(ev.geometry)
    c = K.Context(0)
    try:
        max_len = 18
        st, cov, q, _ = c.make_seeds(t["hit_offsets"], t["hit_valid"], t["hit_pos"], ev.geometry.bz,
                                     0 if name == "align20" else 1)
        ck = torch.empty(28, n * K.n_checkpoint_segments(max_len, seg), dtype=dtype, device=dev)
        out = c.fit_tracks(st, cov, q, *hits, geom, checkpoints=ck, seg=seg, max_len=max_len)
        gs, gh, ga = c.fit_adjoint(st, cov, q, *hits, geom, ck, seg, max_len, out["status"])
        torch.cuda.synchronize()
    finally:
        c.close()
    f = lambda x: x.double().cpu().numpy()
    gs, gh, ga = f(gs).T, f(gh), f(ga)
    off, valid = ev.hit_offsets, ev.hit_valid.astype(bool)
    for k in range(n):
        assert not gh[:, off[k] + max_len:off[k + 1]].any()
    assert not gh[:, ~valid].any()
    assert np.isfinite(gh).all() and np.isfinite(gs).all()
    if dtype == torch.float32:
        return
    tr = truncate(ev, np.full(n, max_len))
    il = [(i, j) for i in range(6) for j in range(i + 1)]
    C0 = np.zeros((n, 6, 6))
    for k, (i, j) in enumerate(il):
        C0[:, i, j] = C0[:, j, i] = f(cov)[k]
    _, os_, oh, oa, _ = O.fit_gradients(torch.tensor(f(st).T), torch.tensor(C0),
                                        torch.tensor(q.cpu().numpy().astype(np.float64)), tr.hit_offsets, tr.hit_layer,
                                        tr.hit_valid, torch.tensor(tr.hit_pos), tr.hit_cov, tr.geometry)
    os_, oh, oa = os_.numpy(), oh.numpy(), oa.numpy()
    toff = tr.hit_offsets
    for k in range(n):
        a, b = oh[:, toff[k]:toff[k + 1]], gh[:, off[k]:off[k] + toff[k + 1] - toff[k]]
        assert np.linalg.norm(b - a) <= 1e-6 * np.linalg.norm(a), k
        assert np.linalg.norm(gs[k] - os_[k]) <= 1e-5 * np.linalg.norm(os_[k]), k
    assert np.linalg.norm(ga - oa) <= 1e-8 * np.linalg.norm(oa)
