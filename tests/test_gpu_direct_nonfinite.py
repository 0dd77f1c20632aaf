"""Direct model with a profile sample that is not finite (rr_set_profile takes
device samples as they are): every in-transit flux is not finite, as
rr_evaluate's, wherever the sample lies and whichever bins the planet's limb
crosses."""

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

GRID = dict(zcut=0.7, nzin=20, nzlimb=30, ng=96, nk=24, k0=0.01, k1=0.3)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("sample", [0, 25, 49])
def test_no_finite_flux_in_transit(value, sample):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    mu = np.linspace(0.0, 1.0, 50)
    prof = wl.profile_power2(mu, 0.6, 0.6)[None]
    pv = np.array([[0.0, 4.0, 8.0, b, 0.0, 0.0, k] for b in (0.0, 0.5, 0.95)
                   for k in (0.012, 0.1, 0.29)])
    times = np.linspace(-0.3, 0.3, 700)
    tab, ser = rr.Tables(mu, prof, GRID), rr.TimeSeries(times)
    transit = {p: (rr.evaluate_direct(tab, ser, pv, p) < 1.0).cpu().numpy()
               for p in ("fp64", "mixed")}
    bad = prof.copy()
    bad[0, sample] = value
    tab.set_profile(torch.as_tensor(bad, device="cuda"))
    for p, tr in transit.items():
        assert tr.any(axis=1).all()
        for f in (rr.evaluate(tab, ser, pv, p), rr.evaluate_direct(tab, ser, pv, p)):
            f = f.cpu().numpy()
            assert not np.isfinite(f[tr]).any()
            # exposures at first and last contact overlap by less than a rounding of the flux
            assert np.all(f[~tr & np.isfinite(f)] == 1.0)
