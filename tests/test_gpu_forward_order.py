"""The per-tile forward kernel takes its workgroups in an order that depends on
the launch's size (runs of 1, 64 or 256 rows, the rows of one tile before the
next tile): every exposure of every row has to be evaluated whatever the order.
Seven distinct rows are repeated over row counts below, at and above a run's
length and the launch sizes where the rule changes (six tiles: 4096 rows are
24 576 workgroups), with and without supersampling; the seven rows are checked
against the oracle, to the contract's 1e-9 (FP64) and 1e-6 (mixed), and each
repetition against the first, bit for bit."""

import numpy as np
import pytest

import workloads as wl
from oracle import roadrunner as orr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nss", [1, 3])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-9), ("mixed", 1e-6)])
def test_every_order(nss, precision, tol):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    w = wl.population(npv=7, npt=2563)
    exptime = 0.02 if nss > 1 else 0.0
    tab = rr.Tables(w["mu_s"], w["I_s"], wl.TEST_GRID)
    ser = rr.TimeSeries(w["times"], nss=[nss], exptimes=[exptime])
    ref = orr.evaluate(orr.Tables(w["mu_s"], w["I_s"], **wl.TEST_GRID), w["times"], w["pv"],
                       nss=[nss], exptimes=[exptime])
    assert (ref < 1.0).any(axis=1).sum() >= 4
    for npv in (1, 63, 64, 65, 256, 257, 4096, 4097, 4161, 4353):
        print(f"forward order {precision} nss {nss} rows {npv}", flush=True)
        pv = np.tile(w["pv"], (npv // 7 + 1, 1))[:npv]
        got = rr.evaluate_unregistered(tab, ser, pv, precision)
        few = got[:7].cpu().numpy().astype(np.float64)
        assert np.abs(few - ref[:npv]).max() <= tol
        assert torch.equal(got, got[:7].repeat(npv // 7 + 1, 1)[:npv])
    ser.close()
    tab.close()
