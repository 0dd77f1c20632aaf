"""The device's sine and cosine of an angle of a few radians (sincos_near),
built for the host, against mpmath over |x| <= (pi + 2)/2, the largest angle
the Kepler solve hands it.  Bounds: the reduced angle is rounded twice (half an
ulp of 0.79 each) and the result once (half an ulp of 1), the polynomials'
inner roundings add less than one more half ulp and their truncation less than
2e-9 of an ulp's scale: 2.7 half ulps of 1, that is 1.6e-7 and 3e-16."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

mp = pytest.importorskip("mpmath")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("sincos") / "libsincos.so")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-host-only",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2009_08500_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "sincos_probe.hip"), "-o", out],
                   check=True, capture_output=True)
    return ctypes.CDLL(out)


@pytest.mark.parametrize("ctype,name,tol", [(ctypes.c_float, "probe_sincos_near_f", 1.6e-7),
                                            (ctypes.c_double, "probe_sincos_near_d", 3e-16)])
def test_sincos_near(lib, ctype, name, tol):
    fn = getattr(lib, name)
    fn.argtypes = [ctype, ctypes.POINTER(ctype), ctypes.POINTER(ctype)]
    fn.restype = None
    end = (np.pi + 2.0) / 2.0
    edges = np.array([n * np.pi / 4 + d for n in range(-3, 4) for d in (-1e-7, 0.0, 1e-7)])
    s, c = ctype(), ctype()
    with mp.workdps(40):
        for x in np.concatenate([np.linspace(-end, end, 4001), edges]):
            x = ctype(x).value
            fn(x, ctypes.byref(s), ctypes.byref(c))
            assert abs(s.value - mp.sin(x)) <= tol, x
            assert abs(c.value - mp.cos(x)) <= tol, x
    fn(0.0, ctypes.byref(s), ctypes.byref(c))
    assert (s.value, c.value) == (0.0, 1.0)
    fn(float("nan"), ctypes.byref(s), ctypes.byref(c))
    assert s.value != s.value and c.value != c.value
