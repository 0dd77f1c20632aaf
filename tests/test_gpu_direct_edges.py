"""The direct model's row kernel evaluates only the annulus edges that the
planet's limb crosses, 64 grazing nodes and four waves to a workgroup:
against the oracle (which evaluates every edge) at the edges of those ranges:
the smallest grids, node counts around the workgroup's 64, a thousand bins,
planets inside one annulus, on an edge, and as large as the star, central and
grazing.  Bounds are the contract's: 1e-9 (FP64) and 1e-6 (mixed) of the flux.
"""

import numpy as np
import pytest

import workloads as wl
from oracle import roadrunner as orr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    return rr


@pytest.mark.parametrize("nzin,nzlimb,ng", [(1, 1, 2), (1, 3, 64), (20, 30, 65), (5, 2, 128),
                                            (300, 700, 193)])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-9), ("mixed", 1e-6)])
def test_edge_ranges(rr, nzin, nzlimb, ng, precision, tol):
    grid = dict(zcut=0.8, nzin=nzin, nzlimb=nzlimb, ng=ng, nk=2, k0=0.05, k1=0.1)
    edge = 0.8 / nzin                              # an annulus edge
    ks = np.array([1e-3, 0.0123, 0.1, min(1.0, edge), min(1.0, 0.5 * edge), 0.499, 0.5, 0.999, 1.0])
    pv = np.zeros((2 * ks.size, 7))
    pv[:, 1], pv[:, 2] = 5.0, 10.0
    pv[:, 6] = np.tile(ks, 2)
    pv[ks.size:, 3] = 0.7
    mu = np.linspace(0.0, 1.0, 60)
    prof = wl.profile_power2(mu, 0.7, 0.6)
    times = np.linspace(-0.2, 0.2, 333)            # through the centre and both contacts
    ref = orr.evaluate_direct(orr.Tables(mu, prof, **grid), times, pv)
    got = rr.evaluate_direct(rr.Tables(mu, prof, grid), rr.TimeSeries(times), pv,
                             precision).cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= tol
    assert (ref < 1.0).any(axis=1).all()
