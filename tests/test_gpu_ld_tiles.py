"""Per-row limb-darkening tables and their transpose at the edges of their
work split: node counts that are not a multiple of 64, of 16 or of 4 (no
16-byte loads), few bins, row counts around a tile of 16, k-grids for which
fewer than four waves place the sorted rows, k clustered on one k-row, on the
boundary of two, and spread, and impact parameters for which the lowest nodes
are left out (grazing and central).  Fluxes and gradients against the oracle:
1e-9 (FP64) and 1e-6 (mixed) of the flux, the log-likelihood tests' 1e-7 of
the largest gradient component in FP64.
"""

import numpy as np
import pytest

import workloads as wl
from oracle import gradient as ogr
from oracle import roadrunner as orr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    return rr


def inputs(npv, spread, seed):
    rng = np.random.default_rng(seed)
    pv = np.zeros((npv, 7))
    pv[:, 1], pv[:, 2] = 4.0, rng.uniform(5.0, 12.0, npv)
    pv[:, 3] = rng.choice([0.0, 0.3, 0.85, 1.05], npv)
    pv[:, 4] = rng.choice([0.0, 0.3, 0.8], npv)
    pv[:, 5] = rng.uniform(0.0, 2.0 * np.pi, npv)
    pv[:, 6] = 0.1 + spread * rng.uniform(-0.5, 0.5, npv)
    pv[:, 4] = np.where(pv[:, 2] * (1 - pv[:, 4]) > 2.0, pv[:, 4], 0.0)
    mu = np.linspace(0.0, 1.0, 40)
    prof = np.stack([wl.profile_power2(mu, c, a) for c, a in
                     zip(rng.uniform(0.5, 0.8, npv), rng.uniform(0.4, 0.8, npv))])
    return pv, mu, prof[:, None, :]


@pytest.mark.parametrize("ng,nzin,nzlimb,nk,npv,spread", [
    (64, 3, 4, 4, 1, 0.0), (97, 10, 12, 16, 17, 1e-3), (100, 20, 30, 24, 16, 0.15),
    (66, 1, 1, 1100, 33, 0.15), (132, 7, 9, 2100, 15, 1e-4), (193, 40, 61, 60, 50, 0.02)])
def test_fluxes(rr, ng, nzin, nzlimb, nk, npv, spread):
    grid = dict(zcut=0.8, nzin=nzin, nzlimb=nzlimb, ng=ng, nk=nk, k0=0.01, k1=0.3)
    pv, mu, prof = inputs(npv, spread, ng)
    times = np.linspace(-0.5, 4.4, 1500)
    ref = orr.evaluate_ld(orr.Tables(mu, prof[0], **grid), times, pv, prof)
    tab, ser = rr.Tables(mu, prof[0], grid), rr.TimeSeries(times)
    for prec, tol in (("fp64", 1e-9), ("mixed", 1e-6)):
        got = rr.evaluate_ld(tab, ser, pv, prof, prec).cpu().numpy().astype(np.float64)
        assert np.abs(got - ref).max() <= tol, (prec, np.abs(got - ref).max())


@pytest.mark.parametrize("ng,nk,npv,spread", [(64, 4, 1, 0.0), (97, 16, 17, 1e-3),
                                              (100, 24, 35, 0.15), (132, 2100, 16, 1e-4)])
def test_profile_gradients(rr, ng, nk, npv, spread):
    grid = dict(zcut=0.8, nzin=21, nzlimb=30, ng=ng, nk=nk, k0=0.01, k1=0.3)
    pv, mu, prof = inputs(npv, spread, ng)
    pv[:, 3] = np.minimum(pv[:, 3], 0.85)            # every row transits
    rng = np.random.default_rng(5)
    times = np.sort(rng.uniform(-0.3, 0.3, 400))
    obs = 1.0 - 0.01 * rng.uniform(0.0, 1.0, 400)
    tab, ser = rr.Tables(mu, prof[0], grid), rr.TimeSeries(times)
    ll, g, gp = [x.cpu().numpy() for x in
                 rr.loglik_grad_ld(tab, ser, pv, prof, obs, 1e-3, "fp64")]
    otab = orr.Tables(mu, prof[0], **grid)
    for i in range(0, npv, 5):
        oll, og, ogp = ogr.loglik_grad(orr.with_profile(otab, prof[i]), times, pv[i:i + 1], obs,
                                       1e-3)
        np.testing.assert_allclose(ll[i], oll[0], rtol=1e-11)
        assert np.abs(g[i] - og[0]).max() <= 1e-7 * np.abs(og[0]).max()
        assert np.abs(gp[i] - ogp).max() <= 1e-7 * np.abs(ogp).max()
