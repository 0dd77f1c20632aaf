"""How librr.so launches the log-likelihood kernel, run by
tests/test_loglik_plan_cpu.py in a child process with hip_recorder.cpp
preloaded (no GPU: a device of 256 CUs with 160 KiB of LDS per workgroup).

Usage: python loglik_plan_calls.py <librr.so> <path of _lib.py> lds|parts
"""

import ctypes
import importlib.util
import sys

import numpy as np

LDS = 160 << 10
STATIC = 512                       # what the kernel declares itself, at most


def main(lib_path, lib_py, what):
    spec = importlib.util.spec_from_file_location("rr_lib_decls", lib_py)
    decl = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(decl)
    rec = ctypes.CDLL(None)
    L = ctypes.CDLL(lib_path)
    decl._declare(L)

    def p(a):
        return a.ctypes.data_as(ctypes.c_void_p)

    mu = np.linspace(0.0, 1.0, 20)
    buf = np.zeros(1 << 20)        # stands for every device array: nothing reads it
    d = p(buf)

    def tables(npb, ng):
        grid = decl.RRGrid(0.7, 10, 10, ng, 8, 0.01, 0.3)
        tab, prof = ctypes.c_void_p(), np.ones((npb, 20))
        assert L.rr_prepare_ld(p(mu), p(prof), 20, npb, ctypes.byref(grid), ctypes.byref(tab)) == 0
        return tab

    def kernel(tab, npb, npv, npt, nss, precision, profile):
        """(workgroups, dynamic LDS) of the launch with the most LDS."""
        pb, n, ex = np.zeros(1, np.int32), np.full(1, nss, np.int32), np.zeros(1)
        first = rec.recorder_size()
        rc = L.rr_loglik_grad(tab, d, None, npt, p(pb), p(n), p(ex), 1, d, npv, 6 + npb, precision,
                              d, 1.0, None, d, d, d if profile else None, None)
        assert rc == 0, L.rr_last_error()
        out = []
        for i in range(first, rec.recorder_size()):
            blocks, lds = ctypes.c_long(), ctypes.c_long()
            rec.recorder_launch(i, ctypes.byref(blocks), ctypes.byref(lds))
            out.append((lds.value, blocks.value))
        lds, blocks = max(out)
        return blocks, lds

    def resident(lds):
        return min(4, LDS // (lds + STATIC))

    if what == "lds":
        kept = 0
        for npb, ng in ((1, 96), (1, 512), (2, 512), (4, 96), (4, 192), (4, 512), (5, 192),
                        (8, 96), (8, 192), (8, 512), (16, 96), (16, 256)):
            tab = tables(npb, ng)
            _, none = kernel(tab, npb, 100, 5000, 11, decl.RR_FP64, True)   # more than are kept
            for nss in (1, 5, 10):
                _, lds = kernel(tab, npb, 100, 5000, nss, decl.RR_FP64, True)
                assert lds >= none and lds + STATIC <= LDS, (npb, ng, nss, lds)
                assert 2 * resident(lds) > resident(none), (npb, ng, nss, lds, none)
                kept += lds > none
            L.rr_free_tables(tab)
        assert kept >= 24, kept
    else:
        tab = tables(1, 96)
        for precision, waves in ((decl.RR_FP64, 2048), (decl.RR_MIXED, 4096)):
            for profile in (False, True):
                for npv in (60, 100, 200, 256):        # no part of a second round
                    blocks, _ = kernel(tab, 1, npv, 50000, 5, precision, profile)
                    # (at most one for 32 time blocks of 64, with the profile gradient 16)
                    parts = min(waves // (2 * npv), 25, 16 if profile else 25)
                    assert blocks == npv * parts and 2 * blocks <= waves, (npv, blocks)
                blocks, _ = kernel(tab, 1, 300, 50000, 5, precision, profile)
                assert blocks == 300 * -(-waves // 600), blocks
                assert kernel(tab, 1, 5000, 50000, 5, precision, profile)[0] == 5000
    print("OK")


if __name__ == "__main__":
    main(*sys.argv[1:])
