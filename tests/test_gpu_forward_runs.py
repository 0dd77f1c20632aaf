"""Runs of rows in the per-tile forward launch (balanced lengths, the last one
shorter, more runs than one grid dimension holds): every row is evaluated once,
bit for bit as the same row in a small call."""

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npv,npt,nss", [
    (258, 2563, 3), (300, 700, 1), (513, 40, 2),      # two and three runs, not of equal length
    (70001, 30, 3),                                   # row by row: runs in the third dimension
    (65535 * 64 + 3, 9, 1)])                          # the same at 64 rows
def test_every_row(npv, npt, nss):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    w = wl.population(npv=11, npt=10)
    pv = w["pv"].copy()
    pv[:, 0] = 0.0
    tab = rr.Tables(w["mu_s"], w["I_s"], wl.TEST_GRID)
    ser = rr.TimeSeries(np.linspace(-0.2, 0.2, npt), nss=[nss], exptimes=[0.01 if nss > 1 else 0.0])
    ref = rr.evaluate_unregistered(tab, ser, pv, "mixed")
    assert bool((ref < 1.0).any(dim=1).all())
    idx = torch.arange(npv, device="cuda") % 11
    rows = torch.as_tensor(pv, device="cuda")[idx].contiguous()
    got = rr.evaluate_unregistered(tab, ser, rows, "mixed")
    assert torch.equal(got, ref[idx])
