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


def test_bench_inner_points_match_the_library(tmp_path):
    """bench.py prices the interior's launch with its own count of the inner region, which must be the library's."""
    import bench

    cases = [(n, cp, st) for n in ((512, 512, 512), (480, 460, 456), (261, 243, 197), (611, 387, 453), (97, 200, 640),
                                   (129, 250, 512), (300, 300, 300), (64, 1024, 300))
             for cp in ((20,) * 6, (10, 12, 9, 20, 15, 11), (0, 20, 20, 0, 0, 20), (0,) * 6) for st in (0, 1)
             if n[0] * n[1] * n[2] >= (16000000 if st else 12000000)]
    line = []
    for n, cp, st in cases:
        deep = st == 0 and n[0] * n[1] * n[2] >= 100000000
        line.append(" ".join(map(str, n + cp + (64 if st else 32, 16 if deep else 8))))
    out = subprocess.run([_build(tmp_path), "inner"], input="\n".join(line), check=True, capture_output=True, text=True,
                         timeout=60)
    got = [int(v) for v in out.stdout.split()]
    assert max(got) > 0 and got == [bench.inner_points(*c) for c in cases]
