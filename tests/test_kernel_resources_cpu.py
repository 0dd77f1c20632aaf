"""Registers of the kernels whose time depends on the waves that a SIMD holds:
compiled for gfx950 as the library is, each keeps at least the waves per SIMD
that its launch is planned for and spills nothing.
"""

import importlib.util
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2009_08500_amd", "csrc")

# source, kernel -> waves per SIMD
WAVES = {
    "rr_forward.hip": {
        **{f"k_forward<double, true, {j}>": 4 for j in (4, 8, 16)},
        **{f"k_forward<float, true, {j}>": 7 for j in (4, 8)},
        "k_forward_split<double, true, false>": 3,
        "k_forward_split<float, true, false>": 5,
    },
    # <real, one passband, profile gradient>
    "rr_adjoint.hip": {
        **{f"k_adjoint<double, {one}, {prof}>": 2 for one in ("true", "false")
           for prof in ("true", "false")},
        **{f"k_adjoint<float, {one}, {prof}>": 4 for one in ("true", "false")
           for prof in ("true", "false")},
    },
}


def resources(source, tmp_path):
    spec = importlib.util.spec_from_file_location(
        "rr_build", os.path.join(ROOT, "paper_2009_08500_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    r = subprocess.run([hipcc, *build.HIPCC_FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(CSRC, source), "-o", str(tmp_path / "x.o")],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr
    found = re.findall(r"remark:.*?(Function Name|Occupancy \[waves/SIMD\]|VGPRs Spill): (\S+)",
                       r.stderr)
    names = [v for k, v in found if k == "Function Name"]
    plain = subprocess.run([shutil.which("c++filt") or "/opt/rocm/llvm/bin/llvm-cxxfilt"],
                           input="\n".join(names), capture_output=True, text=True).stdout.split("\n")
    out, it = {}, iter(plain)
    for key, value in found:
        if key == "Function Name":
            m = re.search(r"(k_\w+(?:<[^()]*>)?)\(", next(it).replace("(anonymous namespace)::", ""))
            cur = out.setdefault(m.group(1) if m else value, {})
        else:
            cur[key] = int(value)
    return out


@pytest.mark.parametrize("source", sorted(WAVES))
def test_waves_per_simd(source, tmp_path):
    got = resources(source, tmp_path)
    for kernel, waves in WAVES[source].items():
        r = got[kernel]
        assert r["Occupancy [waves/SIMD]"] >= waves, (kernel, r)
        assert r["VGPRs Spill"] == 0, (kernel, r)
