"""The split launch over large populations: transit and streaming workgroups
alternate where the transits alone would fill the chip, and an output beyond
256 MB is stored past the caches.  Just above both lines, with whole and ragged
rows and an invalid row among them: seven distinct rows repeated over the
population, each repetition equal to the seven rows' own call bit for bit (its
launch is plain), and that call within the contract's 1e-9 (FP64) and 1e-6
(mixed) of the oracle."""

import numpy as np
import pytest

import workloads as wl
from oracle import roadrunner as orr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npv,npt,precision", [
    (5121, 5000, "mixed"), (5125, 5003, "mixed"),       # alternating order
    (3073, 5000, "fp64"), (3077, 5001, "fp64"),
    (1400, 50000, "mixed"), (1345, 49999, "mixed"),     # beyond the caches too
    (701, 50000, "fp64"), (4099, 8200, "fp64")])
def test_large_population(npv, npt, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    print(f"split large {precision} {npv} x {npt}", flush=True)
    w = wl.population(npv=7, npt=npt)
    w["pv"][4, 6] = 0.9                                  # outside the tables
    tab = rr.Tables(w["mu_s"], w["I_s"], wl.TEST_GRID)
    ser = rr.TimeSeries(w["times"])
    assert ser.kernel(tab, npv, precision) == "split"
    assert ser.kernel(tab, 7, precision) == "split_fused"
    pv = np.tile(w["pv"], (npv // 7 + 1, 1))[:npv]
    got = rr.evaluate(tab, ser, pv, precision)
    few = rr.evaluate(tab, ser, w["pv"], precision)
    ref = orr.evaluate(orr.Tables(w["mu_s"], w["I_s"], **wl.TEST_GRID), w["times"], w["pv"])
    ok = [r for r in range(7) if r != 4]
    assert bool(few[4].isnan().all()) and np.isnan(ref[4]).all()
    tol = 1e-9 if precision == "fp64" else 1e-6
    assert np.abs(few[ok].cpu().numpy().astype(np.float64) - ref[ok]).max() <= tol
    assert (ref[ok] < 1.0).any(axis=1).all()
    # as whole numbers, so that NaN rows compare too
    bits = torch.int64 if precision == "fp64" else torch.int32
    for r in range(7):
        rows = got[r::7].view(bits)
        assert bool((rows == few[r].view(bits)).all()), r
    ser.close()
    tab.close()
