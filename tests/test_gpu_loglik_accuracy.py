"""logL in FP64 of data whose noise is far below the transit depth: it is a
sum of N small squares, so its relative error is a few roundings of that sum
and what the roundings of the fluxes give.  The reference is the exactly
rounded sum (math.fsum) over the forward kernel's FP64 fluxes; with fluxes
that differ by at most dF (8 half-ulps of 1) in n of the N exposures,

    |d logL / logL| <= sum |r| dF / (sum r^2 / 2) <= 2 dF sqrt(n / N) / rms(r)

by Cauchy and Schwarz, and 1e-14 for the sum itself.
"""

import math

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

GRID = dict(zcut=0.7, nzin=20, nzlimb=30, ng=128, nk=24, k0=0.5, k1=0.95)
SIGMA = 20e-6


@pytest.fixture(scope="module")
def rr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    return rr


@pytest.mark.parametrize("npv,npt,nss,shuffle,profile", [
    (1, 20000, 1, False, False), (3, 20000, 5, True, True), (300, 9001, 1, True, False),
    (2100, 4097, 1, False, False)])
def test_small_noise(rr, npv, npt, nss, shuffle, profile):
    rng = np.random.default_rng(npt)
    pv = np.zeros((npv, 7))
    pv[:, 1], pv[:, 2] = 3.0, 10.0
    pv[:, 3] = 0.2 + 1e-9 * np.arange(npv)
    pv[:, 6] = 0.8
    times = np.sort(rng.uniform(-1.0, 7.0, npt))
    if shuffle:
        times = rng.permutation(times)
    mu = np.linspace(0.0, 1.0, 60)
    tab = rr.Tables(mu, wl.profile_power2(mu, 0.6, 0.6)[None], GRID)
    ser = rr.TimeSeries(times, nss=[nss], exptimes=[0.001])
    flux = rr.evaluate_unregistered(tab, ser, pv[:min(npv, 5)], "fp64").cpu().numpy()
    obs = flux[0] + SIGMA * rng.standard_normal(npt)
    ll = rr.loglik_grad(tab, ser, pv, obs, SIGMA, "fp64", profile=profile)[0].cpu().numpy()
    n = int((flux[0] < 1.0).sum())
    tol = 2.0 * 8 * 2.0 ** -53 * math.sqrt(n / npt) / SIGMA + 1e-14
    for i, f in enumerate(flux):
        ref = math.fsum((-0.5 * ((obs - f) / SIGMA) ** 2).tolist())
        assert abs(ll[i] / ref - 1.0) <= tol, (abs(ll[i] / ref - 1.0), tol)
