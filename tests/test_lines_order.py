"""The lanes of a wave hand their results to each other through LDS on the way out (csrc/kernels_lines.h): what they stage is read by other lanes, so the
compiler may move no read before the stores of its pass and no store of the next pass before the reads.  Checked in the code that the compiler is left
with (its intermediate form, at the library's optimisation level): a fence that it may move no memory access across stands between them."""
import os
import re
import subprocess

import pytest

from paper_2105_04663_amd.build import HIP_FLAGS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("lines") / "check.ll")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    build = subprocess.run([hipcc] + HIP_FLAGS + ["-x", "hip", "--offload-device-only", "-emit-llvm", "-S", os.path.join(ROOT, "tests", "lines_order_check.hip"), "-o", out],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    with open(out) as f:
        return {m.group(1): m.group(0) for m in re.finditer(r"^define [^\n]*?(check_kernel\w*).*?^}", f.read(), re.S | re.M)}


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


def test_reads_and_stores_of_a_pass_are_apart(kernels):
    assert len(kernels) == 5
    for name, body in kernels.items():
        seen = _accesses(body)
        assert seen.count("W") >= 16 and seen.count("R") >= 8, (name, seen)
        assert re.fullmatch(r"(W+F+R+F+)+", seen), (name, seen)
