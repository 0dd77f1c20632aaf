"""The log-likelihood kernel's route to a row's in-transit exposures: blocks
of 64 exposures found by their time bounds, their flagged exposures packed
into batches of 64.  Against the oracle at the edges of the blocks, for times
in any order, with light curves that alternate within a block, for exposures
with more subsamples than the profile gradient keeps, for tables that leave no
LDS for the packing, and for data that are not finite.

Tolerances are those of the log-likelihood's parity tests: FP64 logL 1e-11
relative and gradients 1e-7 of the largest component (the same arithmetic per
subsample as the oracle's, rounding apart), mixed 1e-6 and 2e-4 (FP32 terms).
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


def rowwise_close(a, b, rel):
    scale = np.abs(b).max(axis=-1, keepdims=True)
    assert np.all(np.abs(a - b) <= rel * scale), np.max(np.abs(a - b) / scale)


def walkers(npv, npt, nss, shuffle, grid=wl.TEST_GRID):
    """Walkers over npt times within 1.5 transit durations of conjunction and
    a few far from it, in time order or shuffled."""
    w = wl.loglik_walkers(npv=npv, npt=max(npt, 2), nss=nss)
    P, t0 = w["truth"][1], w["truth"][0]
    rng = np.random.default_rng(npt)
    t = np.sort(t0 + P * (rng.integers(0, 3, npt) + rng.uniform(-0.06, 0.06, npt)))
    t[::7] += 0.3 * P
    w["times"] = rng.permutation(t) if shuffle else np.sort(t)
    otab = orr.Tables(w["mu_s"], w["I_s"], **grid)
    obs = 1.0 - 1e-3 * rng.uniform(0.0, 1.0, npt)
    return w, otab, obs


@pytest.mark.parametrize("npt,nss,shuffle,precision", [
    (1, 1, False, "fp64"), (63, 2, False, "fp64"), (64, 3, True, "mixed"), (65, 5, True, "fp64"),
    (129, 12, False, "fp64"), (2500, 3, True, "fp64"), (2500, 3, False, "mixed"),
    (9000, 1, True, "mixed")])
def test_block_edges(rr, npt, nss, shuffle, precision):
    w, otab, obs = walkers(5, npt, nss, shuffle)
    tab = rr.Tables(w["mu_s"], w["I_s"], wl.TEST_GRID)
    ser = rr.TimeSeries(w["times"], nss=[nss], exptimes=w["exptimes"])
    ll, g, gp = [x.cpu().numpy() for x in rr.loglik_grad(
        tab, ser, w["pv"], obs, w["sigma"], precision, grad=True, profile=True)]
    if precision == "mixed":
        obs = obs.astype(np.float32).astype(np.float64)
    oll, og, ogp = ogr.loglik_grad(otab, w["times"], w["pv"], obs, w["sigma"], nss=[nss],
                                   exptimes=w["exptimes"])
    rel_ll, rel_g = (1e-11, 1e-7) if precision == "fp64" else (1e-6, 2e-4)
    np.testing.assert_allclose(ll, oll, rtol=rel_ll)
    rowwise_close(g, og, rel_g)
    rowwise_close(gp, ogp, rel_g)


def test_alternating_light_curves_and_bad_ids(rr):
    """Two light curves whose exposures alternate (every block holds both),
    then one id out of range: logL is NaN, the gradients stay."""
    w, _, obs = walkers(4, 1000, 3, True)
    rng = np.random.default_rng(2)
    lcids = rng.integers(0, 2, 1000).astype(np.int32)
    I_s = np.concatenate([w["I_s"], w["I_s"] ** 1.2])
    pv = np.concatenate([w["pv"], 0.9 * w["pv"][:, 6:7]], 1)
    kw = dict(lcids=lcids, pbids=[1, 0], nss=[4, 1], exptimes=[0.02, 0.001])
    otab = orr.Tables(w["mu_s"], I_s, **wl.TEST_GRID)
    tab = rr.Tables(w["mu_s"], I_s, wl.TEST_GRID)
    oll, og, ogp = ogr.loglik_grad(otab, w["times"], pv, obs, w["sigma"], **kw)
    ll, g, gp = [x.cpu().numpy() for x in rr.loglik_grad(
        tab, rr.TimeSeries(w["times"], **kw), pv, obs, w["sigma"], "fp64", profile=True)]
    np.testing.assert_allclose(ll, oll, rtol=1e-11)
    rowwise_close(g, og, 1e-7)
    rowwise_close(gp, ogp, 1e-7)
    out = int(np.argmax(np.abs((w["times"] - pv[0, 0]) / pv[0, 1] % 1.0 - 0.5) < 0.3))
    kw["lcids"] = lcids.copy()
    kw["lcids"][out] = 7                       # an exposure far from transit
    ll, g2, _ = [x.cpu().numpy() for x in rr.loglik_grad(
        tab, rr.TimeSeries(w["times"], **kw), pv, obs, w["sigma"], "fp64", profile=True)]
    assert np.isnan(ll).all()
    rowwise_close(g2, og, 1e-7)


@pytest.mark.parametrize("value,expect", [(np.nan, np.nan), (np.inf, -np.inf),
                                          (-np.inf, -np.inf), (1e200, -np.inf)])
@pytest.mark.parametrize("inside", [False, True])
def test_data_not_finite(rr, value, expect, inside):
    w, _, obs = walkers(3, 700, 2, False)
    ph = np.abs((w["times"] - w["truth"][0]) / w["truth"][1] + 0.5) % 1.0 - 0.5
    at = int(np.argmin(np.abs(ph)) if inside else np.argmax(np.abs(ph)))
    tab = rr.Tables(w["mu_s"], w["I_s"], wl.TEST_GRID)
    ser = rr.TimeSeries(w["times"], nss=[2], exptimes=w["exptimes"])
    _, g0 = [x.cpu().numpy() for x in rr.loglik_grad(tab, ser, w["pv"], obs, w["sigma"],
                                                     "fp64")[:2]]
    obs[at] = value
    ll, g = [x.cpu().numpy() for x in rr.loglik_grad(tab, ser, w["pv"], obs, w["sigma"],
                                                     "fp64")[:2]]
    np.testing.assert_array_equal(ll, np.full(3, expect))
    if not inside:
        np.testing.assert_array_equal(g, g0)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_tables_that_fill_lds(rr, precision):
    """Sixteen passbands with the largest ng whose tables leave less LDS
    than the packing needs: exposures are evaluated where they stand."""
    import torch
    lds = torch.cuda.get_device_properties(0).shared_memory_per_block
    per = 2 * 16 * (8 if precision == "fp64" else 4)
    ng = min(4096, (lds - 512) // per)
    grid = dict(wl.TEST_GRID, ng=int(ng), nk=4, nzin=6, nzlimb=8)
    w, _, obs = walkers(3, 300, 2, True)
    I_s = np.repeat(w["I_s"], 16, 0)
    pv = np.concatenate([w["pv"]] + [w["pv"][:, 6:7]] * 15, 1)
    kw = dict(lcids=None, pbids=[0], nss=[2], exptimes=w["exptimes"])
    tab = rr.Tables(w["mu_s"], I_s, grid)
    otab = orr.Tables(w["mu_s"], I_s, **grid)
    ll, g = [x.cpu().numpy() for x in rr.loglik_grad(
        tab, rr.TimeSeries(w["times"], **kw), pv, obs, w["sigma"], precision)[:2]]
    if precision == "mixed":
        obs = obs.astype(np.float32).astype(np.float64)
    oll, og, _ = ogr.loglik_grad(otab, w["times"], pv, obs, w["sigma"], **kw)
    rel_ll, rel_g = (1e-11, 1e-7) if precision == "fp64" else (1e-6, 2e-4)
    np.testing.assert_allclose(ll, oll, rtol=rel_ll)
    rowwise_close(g, og, rel_g)
