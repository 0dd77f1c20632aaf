"""Which memory librr.so uses for a call's temporaries, by stream handle, run by
tests/test_stream_memory_cpu.py in a child process with hip_recorder.cpp
preloaded (no GPU: allocations and launches are recorded, kernels not run).

Usage: python stream_memory_calls.py <librr.so> <path of _lib.py>
"""

import ctypes
import importlib.util
import sys

import numpy as np

PER_THREAD = 2                     # hipStreamPerThread


def main(lib_path, lib_py):
    spec = importlib.util.spec_from_file_location("rr_lib_decls", lib_py)
    decl = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(decl)
    rec = ctypes.CDLL(None)
    L = ctypes.CDLL(lib_path)
    decl._declare(L)

    def log(first):
        out = []
        for i in range(first, rec.recorder_size()):
            op, st, p = ctypes.c_char(), ctypes.c_void_p(), ctypes.c_void_p()
            rec.recorder_get(i, ctypes.byref(op), ctypes.byref(st), ctypes.byref(p))
            out.append((op.value.decode(), st.value or 0, p.value or 0))
        return out

    mu = np.linspace(0.0, 1.0, 20)
    prof = np.ones((1, 20))
    times = np.linspace(0.0, 1.0, 700)
    pb, nss, ex = np.zeros(1, np.int32), np.full(1, 2, np.int32), np.zeros(1)
    npv, npt, npar = 3, times.size, 7
    buf = np.zeros(1 << 20)        # stands for every device array: nothing reads it

    def p(a):
        return a.ctypes.data_as(ctypes.c_void_p)

    grid = decl.RRGrid(0.7, 10, 10, 32, 8, 0.01, 0.3)
    tab, ser = ctypes.c_void_p(), ctypes.c_void_p()
    assert L.rr_prepare_ld(p(mu), p(prof), 20, 1, ctypes.byref(grid), ctypes.byref(tab)) == 0
    assert L.rr_series_create(p(times), None, npt, p(pb), p(nss), p(ex), 1, ctypes.byref(ser)) == 0
    d, F64 = p(buf), decl.RR_FP64
    head = (tab, d, None, npt, p(pb), p(nss), p(ex), 1, d, npv, npar)
    calls = {
        "rr_evaluate": lambda s: L.rr_evaluate(*head, F64, d, s),
        "rr_evaluate_variant": lambda s: L.rr_evaluate_variant(*head, F64, 1, d, s),
        "rr_evaluate_series": lambda s: L.rr_evaluate_series(tab, ser, d, npv, npar, F64, d, s),
        "rr_evaluate_direct": lambda s: L.rr_evaluate_direct(*head, F64, d, s),
        "rr_evaluate_small_planet": lambda s: L.rr_evaluate_small_planet(*head, 0.02, F64, d, s),
        "rr_evaluate_ld": lambda s: L.rr_evaluate_ld(*head, d, F64, d, s),
        "rr_loglik_grad": lambda s: L.rr_loglik_grad(*head, F64, d, 1.0, None, d, d, d, s),
        "rr_loglik_grad_ld": lambda s: L.rr_loglik_grad_ld(*head, d, F64, d, 1.0, d, d, d, s),
        "rr_loglik_grad_small_planet":
            lambda s: L.rr_loglik_grad_small_planet(*head, 0.02, F64, d, 1.0, d, d, s),
    }
    for name, call in calls.items():
        for stream in (PER_THREAD, 0x1000, 0):
            for k in range(4):
                first = rec.recorder_size()
                assert call(ctypes.c_void_p(stream)) == 0, (name, L.rr_last_error())
                ev = log(first)
                launches = [i for i, e in enumerate(ev) if e[0] == "L"]
                assert launches and all(ev[i][1] == stream for i in launches), (name, ev)
                mem = [e for e in ev if e[0] != "L"]
                if stream == PER_THREAD:
                    # memory of the call alone: taken before, given back behind its launches
                    assert [e[0] for e in mem] == ["m", "f"], (name, k, ev)
                    assert ev[0][0] == "m" and ev[-1] == ("f", stream, ev[0][2]), (name, k, ev)
                    assert ev[0][1] == stream, (name, k, ev)
                elif k > 1:
                    assert not mem, (name, k, ev)           # a kept buffer
        # no host memory for a new stream's entry: an error code, and nothing enqueued
        first = rec.recorder_size()
        rec.recorder_no_memory(1)
        rc = call(ctypes.c_void_p(0x2000))
        rec.recorder_no_memory(0)
        assert rc == decl.RR_ENOMEM and not log(first), (name, rc, log(first))
        assert call(ctypes.c_void_p(0x2000)) == 0, name
        L.rr_free_tables(tab)
        assert L.rr_prepare_ld(p(mu), p(prof), 20, 1, ctypes.byref(grid), ctypes.byref(tab)) == 0
        print(name)
    L.rr_free_tables(tab)
    L.rr_series_free(ser)
    print("OK")


if __name__ == "__main__":
    main(sys.argv[1], sys.argv[2])
