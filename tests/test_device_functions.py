"""Functions of the built device code that are not kernels: only right_update, whose pointer is to global memory.  A
helper that takes LDS and is not inlined would reach it through generic pointers, with bases that can lie before the
LDS aperture."""
import os
import shutil
import subprocess

import pytest

from helpers import ROOT

LIB = os.path.join(ROOT, "paper_2403_01254_amd", "_lib", "librkhsba.so")
TOOLS = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


def functions(code_object):
    """(kernels, other functions) of a device code object: a kernel has a descriptor, its name and ".kd"."""
    table = subprocess.run([os.path.join(TOOLS, "llvm-readelf"), "-sW", code_object], check=True, capture_output=True,
                           text=True).stdout
    rows = [line.split() for line in table.splitlines()]
    names = {kind: {r[7] for r in rows if len(r) == 8 and r[3] == kind} for kind in ("FUNC", "OBJECT")}
    kernels = {f for f in names["FUNC"] if f + ".kd" in names["OBJECT"]}
    return kernels, names["FUNC"] - kernels


def test_device_helpers_are_inlined(tmp_path):
    if not os.path.exists(LIB):
        from paper_2403_01254_amd import build
        build.build()
    if not os.path.exists(os.path.join(TOOLS, "llvm-objdump")):
        pytest.skip("no ROCm LLVM tools")
    copy = str(tmp_path / "lib.so")
    shutil.copy(LIB, copy)
    subprocess.run([os.path.join(TOOLS, "llvm-objdump"), "--offloading", copy], check=True, capture_output=True)
    objects = sorted(str(p) for p in tmp_path.iterdir() if p.name.endswith("gfx950"))
    kernels, others = set(), set()
    for obj in objects:
        k, o = functions(obj)
        kernels |= k
        others |= o
    assert len(kernels) > 50  # (the symbols are there to be looked at)
    assert {f for f in others if "right_update" not in f} == set()
