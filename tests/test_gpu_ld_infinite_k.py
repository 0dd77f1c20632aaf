"""Per-row limb darkening: a row whose k is not finite is an invalid row (NaN
logL and gradient, a zero profile gradient), in a matrix-core tile and row by
row; the other rows' outputs are those of the same call with that row's k
outside the tables instead."""

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

GRID = dict(zcut=0.8, nzin=21, nzlimb=30, ng=100, nk=24, k0=0.01, k1=0.3)


@pytest.fixture(scope="module")
def rr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    return rr


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("spread", [1e-3, 0.28])
@pytest.mark.parametrize("k_bad,k_out", [(np.inf, 1e3), (-np.inf, -1e3), (np.nan, -1e3)])
def test_profile_gradient_is_zero(rr, k_bad, k_out, spread, precision):
    npv = 20
    rng = np.random.default_rng(1)
    pv = np.zeros((npv, 7))
    pv[:, 1], pv[:, 2], pv[:, 3] = 4.0, 8.0, rng.uniform(0.0, 0.6, npv)
    end = 0.3 if k_out > 0 else 0.01                  # the k-row of the bad row's neighbours
    pv[:, 6] = end - np.sign(k_out) * spread * rng.uniform(0.0, 1.0, npv)
    mu = np.linspace(0.0, 1.0, 40)
    prof = np.broadcast_to(wl.profile_power2(mu, 0.6, 0.6), (npv, 1, 40)).copy()
    times = np.sort(rng.uniform(-0.3, 0.3, 400))
    obs = 1.0 - 0.01 * rng.uniform(0.0, 1.0, times.size)
    tab, ser = rr.Tables(mu, prof[0], GRID), rr.TimeSeries(times)
    out = []
    for k in (k_bad, k_out):
        pv[7, 6] = k
        out.append([x.cpu().numpy() for x in
                    rr.loglik_grad_ld(tab, ser, pv, prof, obs, 1e-3, precision)])
        ll, g, gp = out[-1]
        assert np.isnan(ll[7]) and np.isnan(g[7]).all() and np.all(gp[7] == 0.0)
    for a, b in zip(*out):
        assert np.array_equal(a, b, equal_nan=True) and np.isfinite(np.delete(a, 7, 0)).all()
