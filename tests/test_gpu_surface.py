"""GPU parity of the FP64 fits where the surface-frame step changes form: fits
that end on their first or second entry (the 6x6 covariance of the first entry
is returned, checkpointed or carried on), hits whose covariance has no
thickness along the surface normal or a strong correlation with it (updated on
the 6x6 covariance), and barrel-disk changes, in every layout."""
import numpy as np
import pytest
import torch

from oracle import kf_oracle as O
from toygen import generate, truncate, workloads

from parity import (backward_probes, compare_fit, gpu_backward, gpu_fit, ill_conditioned, oracle_backward, oracle_fit,
                    rounded_forward)

pytestmark = pytest.mark.gpu

# the bound of the other FP64 parity tests: relative rounding of some 1e-13
# per step over up to 26 steps, with four orders of magnitude of conditioning
TOL = (1e-8, 1e-8)


@pytest.fixture(scope="module")
def kf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as _kf
    return _kf


def _with_correlation(ev):
    """Every third hit's covariance gains a component along (x, y, z) / r that
    ties the normal to both surface directions (still positive definite)."""
    cov = ev.hit_cov.copy()
    e = np.arange(0, ev.n_hits, 3)
    r = np.hypot(ev.hit_pos[0, e], ev.hit_pos[1, e])
    c, s = ev.hit_pos[0, e] / r, ev.hit_pos[1, e] / r
    v = np.stack([0.02 * c - 0.004 * s, 0.02 * s + 0.004 * c, np.full(e.size, 0.01)])
    k = 0
    for i in range(3):
        for j in range(i + 1):
            cov[k, e] += v[i] * v[j]
            k += 1
    ev.hit_cov = cov
    return ev


@pytest.mark.parametrize("layout", [0, 2, 3, 4])
@pytest.mark.parametrize("name,mode,n,length", [("barrel20", 0, 65, 3), ("mixed26", 1, 257, 26), ("mixed26", 1, 64, 4)])
def test_short_and_mixed_fits(kf, name, mode, n, length, layout):
    print("surface step", name, n, length, layout, flush=True)
    ev = _with_correlation(generate(workloads()[name], n))
    ev = truncate(ev, np.minimum(ev.lengths(), length))
    ref = oracle_fit(ev, torch.float64, mode)
    # tracks cut to too few hits have no seed: their status is the seeding's
    bad = ~np.asarray(O.make_seeds(ev.hit_offsets, ev.hit_valid, ev.hit_pos, ev.geometry.bz, mode=mode)[3])
    bad = bad | ill_conditioned(ev, torch.float64, ref, mode, TOL[0], TOL[1])
    unseeded = bad.copy()
    c = kf.Context(0)
    try:
        c.reserve(n, 26)
        c.set_fit_launch(torch.float64, 64, 0, 1, 1, layout)
        compare_fit(gpu_fit(c, kf, ev, torch.float64, mode), ref, TOL[0], TOL[1], ~bad, geom=ev.geometry)
        fwd = rounded_forward(ref, torch.float64)
        o = oracle_backward(ev, torch.float64, fwd)
        bad = backward_probes(ev, torch.float64, lambda **kw: oracle_backward(ev, torch.float64, fwd, **kw), o, TOL)
        compare_fit(gpu_backward(c, kf, ev, torch.float64, fwd), o, TOL[0], TOL[1], ~(bad | unseeded),
                    geom=ev.geometry)
    finally:
        c.close()


@pytest.mark.parametrize("max_len", [1, 2, 3])
def test_first_entries_and_checkpoints(kf, max_len):
    """max_len entries: the result after the first is the oracle's update of
    the seed's covariance (full rank), and each checkpoint holds the result of
    the fit that ends there, bit for bit."""
    ev = _with_correlation(generate(workloads()["barrel20"], 130))
    dt, dev, n = torch.float64, torch.device("cuda", 0), 130
    t = kf.event_tensors(ev, dt, dev)
    geom = kf.Geometry.from_toy(ev.geometry)
    hits = (t["hit_offsets"], t["hit_layer"], t["hit_valid"], t["hit_pos"], t["hit_cov"])
    c = kf.Context(0)
    try:
        ck = torch.empty(28, n * 3, dtype=dt, device=dev)
        c.seed_fit_tracks(*hits, geom, 0, checkpoints=ck, seg=1, max_len=4)
        out = c.seed_fit_tracks(*hits, geom, 0, max_len=max_len)
        torch.cuda.synchronize()
        slot = ck[:, (max_len - 1) * n:max_len * n]
        assert torch.equal(slot[:6], out["state"]) and torch.equal(slot[6:27], out["cov"])
        assert torch.equal(slot[27].to(torch.int8), out["charge"])
        ref = O.fit_event(truncate(ev, np.full(n, 3)))
        if max_len == 3:
            Cg = np.zeros((n, 6, 6))
            k = 0
            for i in range(6):
                for j in range(i + 1):
                    Cg[:, i, j] = Cg[:, j, i] = out["cov"][k].cpu().numpy()
                    k += 1
            Co = ref["C"].numpy()
            s = np.sqrt(np.einsum("nii->ni", Co).clip(1e-12))
            assert (np.abs(Cg - Co) / s[:, :, None] / s[:, None, :]).max() < 1e-7
    finally:
        c.close()


def test_hit_without_thickness(kf):
    """A hit covariance that is singular along the normal leaves S singular:
    the 6x6 update takes it and the track stops or carries on as it does
    there, with finite results; its neighbours are not touched."""
    ev = generate(workloads()["barrel20"], 64)
    ref = oracle_fit(ev, torch.float64, 0)
    bad = ill_conditioned(ev, torch.float64, ref, 0, TOL[0], TOL[1])
    e = ev.hit_offsets[10] + 7
    ev.hit_cov[:, e] = 0.0
    c = kf.Context(0)
    try:
        g = gpu_fit(c, kf, ev, torch.float64, 0)
        assert np.isfinite(g["p"]).all() and np.isfinite(g["C"]).all() and np.isfinite(g["chi2"]).all()
        others = ~bad
        others[10] = False
        compare_fit(g, ref, TOL[0], TOL[1], others, geom=ev.geometry)
    finally:
        c.close()
