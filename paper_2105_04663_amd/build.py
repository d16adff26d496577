"""Compile the HIP/C++ sources in csrc/ into libgspmd.so next to this file (gfx950 only)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "build")
LIB = os.path.join(HERE, "libgspmd.so")
CALL = os.path.join(HERE, "_call" + sysconfig.get_config_var("EXT_SUFFIX"))
# (source, object, extra flags); the MFMA kernels' sources are compiled once per operand layout
UNITS = [(os.path.join(CSRC, f"{name}.hip"), f"{name}_l{n}.o", [f"-DGSPMD_TU_LAYOUT={n}"])
         for name in ("dot_mfma", "dot_split", "dot_mid", "dot_pair") for n in range(4)] + [
    (os.path.join(CSRC, "gspmd.hip"), "gspmd.o", []),
    (os.path.join(CSRC, "plan.cpp"), "plan.o", []),
]
# packed-fp32 code generation is switched off: some of its forms have given wrong results on this hardware
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option", "-Wno-inline-asm"]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed building {os.path.basename(cmd[-1])}")
    if verbose and res.stderr:
        sys.stderr.write(res.stderr)


def build(verbose: bool = False, only=None) -> str:
    """Compile every unit (`only`: those whose object name starts so, the other objects being there) and link."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    objects = [os.path.join(OBJ, obj) for _, obj, _ in UNITS]
    cmds = [[hipcc] + HIP_FLAGS + flags + ["-x", "hip", "-c", src, "-o", os.path.join(OBJ, obj)] for src, obj, flags in UNITS
            if only is None or obj.startswith(tuple(only))]
    with ThreadPoolExecutor(max_workers=min(8, int(os.environ.get("MAX_JOBS", "8")))) as pool:
        list(pool.map(lambda c: _run(c, verbose), cmds))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objects + ["-o", LIB + ".tmp"], verbose)
    os.replace(LIB + ".tmp", LIB)
    if only is None:
        try:
            build_call(verbose)
        except (OSError, RuntimeError) as e:      # no C compiler, no Python headers: the binding goes without it
            if os.path.exists(CALL):
                os.remove(CALL)                   # of another build, perhaps of another library
            sys.stderr.write(f"the binding's native entry was not built, calls go through ctypes: {e}\n")
    elif "call" in only:
        build_call(verbose)
    return LIB


def build_call(verbose: bool = False) -> str:
    """The native entry of the binding, for the Python that runs this."""
    cc = os.environ.get("CC", "gcc")
    _run([cc, "-O2", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "call.c"), "-o", CALL + ".tmp"], verbose)
    os.replace(CALL + ".tmp", CALL)
    return CALL


if __name__ == "__main__":
    print(build(verbose=True, only=sys.argv[1:] or None))
