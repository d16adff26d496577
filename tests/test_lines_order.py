"""The lanes of a wave hand their results to each other through LDS on the way out (csrc/kernels_lines.h, dot_mfma_kernel's epilogue): what they stage is read by other lanes, so the
compiler may move no read before the stores of its pass and no store of the next pass before the reads.  Checked in the code that the compiler is left
with (its intermediate form, at the library's optimisation level): a fence that it may move no memory access across stands between them."""
import os
import re
import subprocess

import pytest

from paper_2105_04663_amd.build import HIP_FLAGS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _kernels(source, name, flags, tmp_path):
    """The bodies of the kernels called `name` in a source file, by their mangled names."""
    out = str(tmp_path / "check.ll")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    build = subprocess.run([hipcc] + HIP_FLAGS + flags + ["-x", "hip", "--offload-device-only", "-emit-llvm", "-S", os.path.join(ROOT, source), "-o", out], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    with open(out) as f:
        return {m.group(1): m.group(0) for m in re.finditer(r"^define [^\n]*?(%s\w*).*?^}" % name, f.read(), re.S | re.M)}


def _accesses(body):
    """W, R for a store to and a load from LDS, F for a fence, in the order of the code."""
    seen = ""
    for line in body.splitlines():
        if re.search(r"\bstore [^\n]*addrspace\(3\)", line):
            seen += "W"
        elif re.search(r"= load [^\n]*addrspace\(3\)", line):
            seen += "R"
        elif 'asm sideeffect "", "~{memory}"' in line or re.search(r"\bfence ", line):
            seen += "F"
    return seen


def test_whole_line_stores(tmp_path):
    kernels = _kernels("tests/lines_order_check.hip", "check_kernel", [], tmp_path)
    assert len(kernels) == 5
    for name, body in kernels.items():
        seen = _accesses(body)
        assert seen.count("W") >= 16 and seen.count("R") >= 8, (name, seen)
        assert re.fullmatch(r"(W+F+R+F+)+", seen), (name, seen)


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
def test_dot_mfma_kernel(tmp_path, layout):
    kernels = _kernels("paper_2105_04663_amd/csrc/dot_mfma.hip", "dot_mfma_kernel", [f"-DGSPMD_TU_LAYOUT={layout}"], tmp_path)
    assert len(kernels) == 4
    for name, body in kernels.items():
        seen = _accesses(body.rsplit("@llvm.amdgcn.s.barrier", 1)[1])          # behind the last barrier: the epilogue
        assert seen.count("W") >= 32 and seen.count("R") >= 16, (name, seen)
        assert re.fullmatch(r"F*(W+F+R+F*)+", seen) and "RW" not in seen, (name, seen)
