"""The box lists of the tile kernels, checked by brute force on random sets of
grids (host code only: csrc/tile_host.hpp, compiled with hipcc for the host)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SANITIZE = ["-O1", "-g", "-fno-omit-frame-pointer", "-Xarch_host", "-fsanitize=address", "-Xarch_host",
            "-fsanitize=undefined"]


def _build(tmp_path, flags=("-O2",)):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "tile_lists_check")
    src = os.path.join(ROOT, "tests", "tile_lists_check.cpp")
    inc = os.path.join(ROOT, "paper_2606_06910_amd", "csrc")
    subprocess.run([hipcc, "-std=c++17", "-I", inc, *flags, "-o", exe, src], check=True, capture_output=True)
    return exe


@pytest.mark.parametrize("flags,cases", [(["-O2"], 600), (SANITIZE, 60)], ids=["plain", "asan-ubsan"])
def test_tile_lists_brute_force(tmp_path, flags, cases):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=1", UBSAN_OPTIONS="halt_on_error=1")
    out = subprocess.run([_build(tmp_path, flags), str(cases)], check=False, capture_output=True, text=True, timeout=300,
                         env=env)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout + out.stderr
    inner, face = (int(v) for v in out.stdout.split()[2:4])
    assert inner > cases and face > cases      # every part was there to be checked
