"""hipStreamPerThread names another stream in every thread: two threads that
call on it with the same tables get their own results, bit for bit those of
the calls made alone."""

import threading
import types

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

PER_THREAD = types.SimpleNamespace(cuda_stream=2)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_two_threads(precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2009_08500_amd as rr
    w = wl.loglik_walkers(npv=60, npt=4000, nss=2)
    tab = rr.Tables(w["mu_s"], w["I_s"], wl.TEST_GRID)
    ser = rr.TimeSeries(w["times"], nss=[2], exptimes=w["exptimes"])
    dt = torch.float64 if precision == "fp64" else torch.float32
    obs = torch.as_tensor(1.0 + w["noise"], device="cuda", dtype=dt)
    prof = torch.as_tensor(np.broadcast_to(w["I_s"], (60, 1, 200)).copy(), device="cuda")
    pv = torch.as_tensor(w["pv"], device="cuda")
    sets = [(pv[:20].contiguous(), prof[:20].contiguous()),
            (pv[20:].contiguous(), prof[20:].contiguous())]

    def calls(rows, profiles, stream):
        return [*rr.loglik_grad(tab, ser, rows, obs, 2e-4, precision, profile=True, stream=stream),
                *rr.loglik_grad_ld(tab, ser, rows, profiles, obs, 2e-4, precision, stream=stream),
                rr.evaluate_unregistered(tab, ser, rows, precision, stream=stream),
                rr.evaluate_ld(tab, ser, rows, profiles, precision, stream=stream),
                rr.evaluate_direct(tab, ser, rows, precision, stream=stream)]

    ref = [calls(*s, None) for s in sets]
    torch.cuda.synchronize()
    out = [[], []]

    def work(i):
        for _ in range(20):
            out[i].append(calls(*sets[i], PER_THREAD))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i in range(2):
        assert len(out[i]) == 20
        for r in out[i]:
            assert all(torch.equal(a, b) for a, b in zip(r, ref[i]))
