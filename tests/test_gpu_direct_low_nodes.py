"""The direct model leaves out the grazing nodes below the smallest separation a
row's orbit can reach: light curves that come closest to that bound, against the
oracle (which tabulates every node), within the contract's 1e-9 (FP64) and 1e-6
(mixed).  Impact parameters from 0 to a grazing 1.05, circular and strongly
eccentric orbits with the transit at periastron and apastron, where the bound is
tight, and on the sides, where it is loose; exposures closely spaced around
mid-transit, where the separation is smallest."""

import numpy as np
import pytest

import workloads as wl
from oracle import roadrunner as orr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ng", [64, 512])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-9), ("mixed", 1e-6)])
def test_closest_separation(ng, precision, tol):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    rows = [(b, e, w, k) for b in (0.0, 0.02, 0.3, 0.77, 1.05)
            for e, w in ((0.0, 0.0), (0.6, np.pi / 2), (0.6, -np.pi / 2), (0.6, 0.0), (0.3, 3.0))
            for k in (0.01, 0.1, 0.9)]
    pv = np.array([[0.0, 6.0, 14.0, b, e, w, k] for b, e, w, k in rows])
    times = np.concatenate([np.linspace(-0.4, 0.4, 401), np.linspace(-1e-3, 1e-3, 101)])
    grid = dict(wl.TEST_GRID, ng=ng)
    mu = np.linspace(0.0, 1.0, 60)
    prof = wl.profile_power2(mu, 0.7, 0.6)
    ref = orr.evaluate_direct(orr.Tables(mu, prof, **grid), times, pv)
    got = rr.evaluate_direct(rr.Tables(mu, prof, grid), rr.TimeSeries(times), pv,
                             precision).cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= tol
    # every row whose planet reaches the disk has a transit among the times
    assert np.array_equal((ref < 1.0).any(axis=1), pv[:, 3] < 1.0 + pv[:, 6])
