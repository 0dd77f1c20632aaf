"""The benchmark's words for what a call launches, and the kernel names it looks
counters up by: the names that the compiled library's kernels have."""

import os
import re

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def compiled_kernels():
    """Kernel names of the source, by its template instantiations' launches."""
    with open(os.path.join(ROOT, "paper_2009_08500_amd", "csrc", "rr_forward.hip")) as fh:
        src = fh.read()
    names = set(re.findall(r"(k_forward_split<(?:float|double), \w+, \w+>)", src))
    for form in re.findall(r"k_forward<R, (\w+, \d+)>", src):
        names |= {f"k_forward<{r}, {form}>" for r in ("float", "double")}
    return names


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("kind,order", [
    ("split_fused", (False, False)), ("split", (False, False)), ("split", (True, False)),
    ("split", (False, True)), ("split", (True, True)), ("tiles", (False, False))])
def test_launch_text(kind, order, precision):
    name, text = bench.forward_kernel(kind, precision, order)
    assert name in compiled_kernels()
    if kind == "split":
        assert name.endswith(", false, true>") == any(order)
    assert ("per-row setup" in text) == (kind != "split_fused")
    assert text.endswith(f"forward kernel '{name}'")
