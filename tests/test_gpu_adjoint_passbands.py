"""Log-likelihood gradients over 2, 5 and 16 passbands whose exposures alternate
within every block: each wave sums d logL / dk and d logL / d I_star per passband
in LDS.  Against the oracle with the parity tests' tolerances (FP64 1e-7 of the
largest component, mixed 2e-4: FP32 terms), and the same bits twice."""

import numpy as np
import pytest

import workloads as wl
from oracle import gradient as ogr
from oracle import roadrunner as orr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,rel", [("fp64", 1e-7), ("mixed", 2e-4)])
@pytest.mark.parametrize("npb", [2, 5, 16])
def test_gradients_per_passband(npb, precision, rel):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    rng = np.random.default_rng(npb)
    w = wl.loglik_walkers(npv=3, npt=10, nss=1)
    t0, P = w["truth"][0], w["truth"][1]
    times = t0 + P * (rng.integers(0, 3, 1500) + rng.uniform(-0.05, 0.05, 1500))
    obs = 1.0 - 1e-3 * rng.uniform(0.0, 1.0, 1500)
    if precision == "mixed":
        obs = obs.astype(np.float32).astype(np.float64)
    I_s = np.concatenate([w["I_s"] ** (0.8 + 0.03 * i) for i in range(npb)])
    pv = np.concatenate([w["pv"][:, :6]] + [w["pv"][:, 6:7] * (1 - 0.01 * i) for i in range(npb)], 1)
    kw = dict(lcids=rng.integers(0, npb, 1500).astype(np.int32), pbids=list(range(npb))[::-1],
              nss=[1 + i % 3 for i in range(npb)], exptimes=[0.002 * (i % 3) for i in range(npb)])
    tab, ser = rr.Tables(w["mu_s"], I_s, wl.TEST_GRID), rr.TimeSeries(times, **kw)
    got = [[x.cpu().numpy() for x in rr.loglik_grad(tab, ser, pv, obs, 2e-4, precision,
                                                    profile=True, istar_grad=True)]
           for _ in range(2)]
    assert all(np.array_equal(a, b) for a, b in zip(*got))
    ref = ogr.loglik_grad(orr.Tables(w["mu_s"], I_s, **wl.TEST_GRID), times, pv, obs, 2e-4,
                          want_istar=True, **kw)
    np.testing.assert_allclose(got[0][0], ref[0], rtol=1e-11 if precision == "fp64" else 1e-6)
    for a, b in zip(got[0][1:], ref[1:]):
        scale = np.abs(b).max(axis=-1, keepdims=True)
        assert np.all(np.abs(a - b) <= rel * scale), np.max(np.abs(a - b) / scale)
