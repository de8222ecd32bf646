"""FP64 fits with hits whose covariance is singular along the surface normal
only, to rounding: the smallest eigenvalue is what is left of s^2 (t t^T + z
z^T) in floating point, of either sign.  S is singular in exact arithmetic, so
the affected track's numbers are arbitrary; they stay finite, the track goes on
or stops with a status, and no other track is touched."""
import numpy as np
import pytest
import torch

from toygen import generate, workloads

from parity import compare_fit, gpu_fit, ill_conditioned, oracle_fit

pytestmark = pytest.mark.gpu
TOL = (1e-8, 1e-8)   # as in the other FP64 parity tests


@pytest.mark.parametrize("layout", [0, 3])
def test_singular_along_the_normal(layout):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_11728_amd import kf as K
    print("thin hits", layout, flush=True)
    n = 256
    ev = generate(workloads()["barrel20"], n)
    ref = oracle_fit(ev, torch.float64, 0)
    bad = ill_conditioned(ev, torch.float64, ref, 0, TOL[0], TOL[1])
    thin = np.arange(0, n, 3)
    e = np.asarray(ev.hit_offsets)[thin] + 7
    x, y = ev.hit_pos[0, e], ev.hit_pos[1, e]
    tx, ty = -y / np.hypot(x, y), x / np.hypot(x, y)
    s2 = 1e-6
    cov = ev.hit_cov.copy()
    cov[:, e] = np.stack([s2 * tx * tx, s2 * tx * ty, s2 * ty * ty, 0 * tx, 0 * tx, s2 + 0 * tx])
    # the smallest eigenvalue's sign is rounding's
    nn = cov[0, e] * ty * ty - 2 * cov[1, e] * tx * ty + cov[2, e] * tx * tx
    assert np.abs(nn).max() < 1e-20 and np.unique(np.sign(nn)).size > 1
    ev.hit_cov = cov
    ctx = K.Context(0)
    try:
        ctx.set_fit_launch(torch.float64, 256, 0, 1, 1, layout)
        g = gpu_fit(ctx, K, ev, torch.float64, 0)
    finally:
        ctx.close()
    for k in ("p", "C", "chi2"):
        assert np.isfinite(g[k]).all(), k
    others = ~bad
    others[thin] = False
    compare_fit(g, ref, TOL[0], TOL[1], others, geom=ev.geometry)
