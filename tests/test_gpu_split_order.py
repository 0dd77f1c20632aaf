"""Which split launch a large population takes (rr_series_order), on both sides of
each line: the alternating order begins at some row count and the stores past
the caches where the output exceeds 256 MB.  Every case of the large-population
test takes the branch it is there for, and one row less or more than a line
changes no bit of a row."""

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


def setup(rr, npt):
    w = wl.population(npv=7, npt=npt)
    return w, rr.Tables(w["mu_s"], w["I_s"], wl.TEST_GRID), rr.TimeSeries(w["times"])


@pytest.mark.parametrize("npv,npt,precision,order", [
    (5121, 5000, "mixed", (True, False)), (5125, 5003, "mixed", (True, False)),
    (3073, 5000, "fp64", (True, False)), (3077, 5001, "fp64", (True, False)),
    (1400, 50000, "mixed", None), (1345, 49999, "mixed", None),
    (701, 50000, "fp64", None), (4099, 8200, "fp64", None)])
def test_large_cases_take_their_branch(rr, npv, npt, precision, order):
    w, tab, ser = setup(rr, npt)
    got = ser.order(tab, npv, precision)
    if order is None:
        assert got[1]                                    # beyond the caches
    else:
        assert got == order
    assert ser.order(tab, 7, precision) == (False, False)         # fused
    assert rr.TimeSeries(w["times"], nss=[2], exptimes=[0.01]).order(tab, npv, precision) == \
        (False, False)                                   # per tile


def same_rows(rr, w, tab, ser, npv, precision):
    import torch
    bits = torch.int64 if precision == "fp64" else torch.int32
    few = rr.evaluate(tab, ser, w["pv"], precision).view(bits)
    got = rr.evaluate(tab, ser, np.tile(w["pv"], (npv // 7 + 1, 1))[:npv], precision).view(bits)
    return all(bool((got[r::7] == few[r]).all()) for r in range(7))


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_both_sides_of_alternating(rr, precision):
    w, tab, ser = setup(rr, 5000)
    lo, hi = 1100, 8192
    assert not ser.order(tab, lo, precision)[0] and ser.order(tab, hi, precision)[0]
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if ser.order(tab, mid, precision)[0] else (mid, hi)
    assert ser.kernel(tab, hi, precision) == "split"
    assert same_rows(rr, w, tab, ser, hi, precision)
    assert same_rows(rr, w, tab, ser, lo, precision)


@pytest.mark.parametrize("npt,precision", [(50000, "mixed"), (49999, "fp64")])
def test_both_sides_of_the_caches(rr, npt, precision):
    w, tab, ser = setup(rr, npt)
    last = (256 << 20) // (npt * (8 if precision == "fp64" else 4))
    assert not ser.order(tab, last, precision)[1]
    assert ser.order(tab, last + 1, precision)[1] == \
        (ser.kernel(tab, last + 1, precision) == "split")
    for npv in (last, last + 1):
        assert same_rows(rr, w, tab, ser, npv, precision)


def test_arguments(rr):
    import ctypes
    from paper_2009_08500_amd import _lib
    w, tab, ser = setup(rr, 100)
    a, b = ctypes.c_int32(5), ctypes.c_int32(5)
    f = _lib.lib().rr_series_order
    assert f(tab.handle, ser.handle, 10, 5, ctypes.byref(a), ctypes.byref(b)) == _lib.RR_EINVAL
    assert f(tab.handle, None, 10, 0, ctypes.byref(a), ctypes.byref(b)) == _lib.RR_EINVAL
    assert f(tab.handle, ser.handle, 10, 0, None, ctypes.byref(b)) == _lib.RR_EINVAL
