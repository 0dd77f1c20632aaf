"""A call's temporaries by stream handle, on the host: on hipStreamPerThread,
one handle for a different stream in every thread, no buffer outlives its call;
and without host memory for a new stream's entry a call returns RR_ENOMEM
(tests/host/stream_memory_calls.py over a recording stand-in for the HIP
runtime)."""

import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2009_08500_amd")


def test_nothing_is_kept_for_the_per_thread_handle(tmp_path):
    gxx, lib = shutil.which("g++"), os.path.join(PKG, "librr.so")
    if not gxx or not os.path.exists(lib) or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("needs g++, the HIP headers and a built librr.so")
    rec = str(tmp_path / "librecorder.so")
    subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(ROOT, "tests", "host", "hip_recorder.cpp"),
                    "-o", rec], check=True, capture_output=True)
    r = subprocess.run([sys.executable,
                        os.path.join(ROOT, "tests", "host", "stream_memory_calls.py"), lib,
                        os.path.join(PKG, "_lib.py")], capture_output=True, text=True,
                       env=dict(os.environ, LD_PRELOAD=rec), timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("OK")
