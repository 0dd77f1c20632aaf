"""A row given the tables' own profile: in FP64 its fluxes, log-likelihood and
gradient are those of the shared tables, bit for bit (the same weights, the
bins added in the same order), for rows in matrix-core tiles (one k-row, two)
and row by row, and for node counts with and without 16-byte rows."""

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    return rr


@pytest.mark.parametrize("ng,nzin,nzlimb,nk,npv,spread", [
    (96, 20, 30, 24, 40, 0.2), (96, 20, 30, 24, 33, 1e-3), (130, 33, 34, 40, 50, 0.008),
    (97, 3, 2, 24, 17, 0.05), (512, 60, 120, 64, 70, 0.004), (64, 1, 1, 1200, 20, 1e-4)])
def test_same_bits(rr, ng, nzin, nzlimb, nk, npv, spread):
    import torch
    grid = dict(zcut=0.7, nzin=nzin, nzlimb=nzlimb, ng=ng, nk=nk, k0=0.01, k1=0.3)
    rng = np.random.default_rng(ng + npv)
    pv = wl.population(npv=npv, npt=10)["pv"]
    pv[:, 0], pv[:, 1] = 0.0, 4.0
    pv[:, 6] = 0.12 + spread * rng.uniform(-0.5, 0.5, npv)
    times = np.sort(rng.uniform(-0.4, 0.4, 3000))
    mu = np.linspace(0.0, 1.0, 50)
    prof = wl.profile_power2(mu, 0.6, 0.6)
    own = np.broadcast_to(prof, (npv, 1, 50)).copy()
    tab, ser = rr.Tables(mu, prof[None], grid), rr.TimeSeries(times)
    assert torch.equal(rr.evaluate_ld(tab, ser, pv, own, "fp64"),
                       rr.evaluate_unregistered(tab, ser, pv, "fp64"))
    obs = 1.0 - 0.01 * rng.uniform(0.0, 1.0, times.size)
    a = rr.loglik_grad_ld(tab, ser, pv, own, obs, 1e-3, "fp64", profile=False)
    b = rr.loglik_grad(tab, ser, pv, obs, 1e-3, "fp64")
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
