"""The log-likelihood's temporaries: kept per stream between calls, one call's
own while it is enqueued, and a graph's own under capture.  Every result is
compared bitwise with the same call made alone (the sums have a fixed order).
"""

import threading

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


def setup(rr, npv=40, npt=4000):
    import torch
    w = wl.loglik_walkers(npv=npv, npt=npt, nss=2)
    tab = rr.Tables(w["mu_s"], w["I_s"], wl.TEST_GRID)
    ser = rr.TimeSeries(w["times"], nss=[2], exptimes=w["exptimes"])
    obs = torch.as_tensor(1.0 + w["noise"], device="cuda")
    pv = torch.as_tensor(w["pv"], device="cuda")
    return tab, ser, pv, obs


def test_sizes_up_and_down_on_two_streams(rr):
    import torch
    tab, ser, pv, obs = setup(rr)
    torch.cuda.synchronize()
    calls = [(n, prof) for n in (3, 40, 1, 17) for prof in (False, True)]
    ref = [[x.clone() for x in rr.loglik_grad(tab, ser, pv[:n], obs, 2e-4, profile=prof)
            if x is not None] for n, prof in calls]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = {}
    for k, (n, prof) in enumerate(calls):
        for i, s in enumerate(streams):
            got[k, i] = rr.loglik_grad(tab, ser, pv[:n], obs, 2e-4, profile=prof, stream=s)
    torch.cuda.synchronize()
    for (k, _), out in got.items():
        for a, b in zip([x for x in out if x is not None], ref[k]):
            assert torch.equal(a, b)


def test_two_threads_on_one_stream(rr):
    """Their calls interleave on the stream, never inside one another."""
    import torch
    tab, ser, pv, obs = setup(rr)
    sets = [pv[:20].contiguous(), pv[20:].contiguous()]
    ref = [[x.clone() for x in rr.loglik_grad(tab, ser, p, obs, 2e-4, profile=True)] for p in sets]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    out = [[], []]

    def work(i):
        for _ in range(40):
            out[i].append(rr.loglik_grad(tab, ser, sets[i], obs, 2e-4, profile=True,
                                         stream=stream))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i in range(2):
        assert len(out[i]) == 40
        for r in out[i]:
            for a, b in zip(r, ref[i]):
                assert torch.equal(a, b)


@pytest.mark.parametrize("warm", [False, True])
def test_capture_owns_its_memory(rr, warm):
    """A captured call, on a stream with or without kept memory, replays to
    the eager result after larger calls on that stream and new rows in place."""
    import torch
    tab, ser, pv, obs = setup(rr)
    rows = pv[:9].clone()
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    if warm:
        rr.loglik_grad(tab, ser, rows, obs, 2e-4, stream=s)
        torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ll, gr, _ = rr.loglik_grad(tab, ser, rows, obs, 2e-4, stream=s)
    for k in (0, 9, 18):
        rows.copy_(pv[k:k + 9])
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        rll, rgr, _ = rr.loglik_grad(tab, ser, pv[k:k + 9].contiguous(), obs, 2e-4)
        assert torch.equal(ll, rll) and torch.equal(gr, rgr)
        rr.loglik_grad(tab, ser, pv, obs, 2e-4, profile=True, stream=s)     # grows the kept memory
        torch.cuda.synchronize()


def test_weights_of_a_broadcast_gradient(rr):
    """backward of logl.sum() (a broadcast gradient), of a weighted sum and of
    a contiguous gradient of equal weights."""
    import torch
    tab, ser, pv, obs = setup(rr, npv=6)
    prof = torch.as_tensor(wl.profile_power2(np.linspace(0, 1, 200), 0.6, 0.6)[None],
                           device="cuda")

    def grads(weigh):
        p = prof.clone().requires_grad_(True)
        q = pv.clone().requires_grad_(True)
        return torch.autograd.grad(weigh(rr.RRLogLik.apply(q, p, tab, ser, obs, 2e-4, "fp64")),
                                   [q, p])

    a = grads(lambda x: x.sum())
    b = grads(lambda x: (x * torch.ones_like(x)).sum())
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    w = torch.arange(1.0, 7.0, dtype=torch.float64, device="cuda")
    c = grads(lambda x: (x * w).sum())
    assert torch.equal(c[0], a[0] * w[:, None])
    d = rr.loglik_grad(tab, ser, pv, obs, 2e-4, grad=False, profile=True, wprof=w)[2]
    assert torch.equal(c[1], d)
