"""CPU check of the index arithmetic of the moves (csrc/kernels_basic.h: division by a precomputed multiplier)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_division_by_multiplication(tmp_path):
    exe = str(tmp_path / "move_index_check")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    build = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-command-line-argument",
                            "-x", "hip", os.path.join(ROOT, "tests", "move_index_check.hip"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert run.returncode == 0 and "move index ok" in run.stdout, run.stdout[-3000:] + run.stderr[-1000:]
