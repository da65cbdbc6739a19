"""The library's host code on the CPU, against a stand-in for the HIP runtime
(hip_stub.cpp) that counts launches and graph instantiations: what a call
enqueues, and what it keeps, where the results alone do not show it."""
import ctypes
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from paper_2606_06910_amd import _lib, build_lib

TESTS = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    """libfdtd built for the host alone and linked with the stand-in."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("host")
    src = [os.path.join(build_lib.CSRC, s) for s in build_lib.SOURCES] + [os.path.join(TESTS, "hip_stub.cpp")]

    def obj(s):
        o = str(d / (os.path.basename(s) + ".o"))
        subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-w", "-I", build_lib.CSRC, "-c", "-o",
                        o, s], check=True, capture_output=True)
        return o

    with ThreadPoolExecutor(4) as ex:
        objs = list(ex.map(obj, src))
    # each object names the embedded device code it was built without
    fat = sorted(set(re.findall(r"__hip_fatbin_\w+", subprocess.run(["nm", "-u"] + objs, check=True, capture_output=True,
                                                                   text=True).stdout)))
    (d / "fat.c").write_text("".join("const unsigned %s[4] = {0};\n" % f for f in fat))
    so = str(d / "libfdtd_host.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-o", so, str(d / "fat.c")] + objs + ["-lstdc++", "-lm"], check=True,
                   capture_output=True)
    L = ctypes.CDLL(so)
    L.stub_launches.restype = L.stub_blocks.restype = L.stub_instantiated.restype = ctypes.c_long
    L.fdtd_last_error.restype = L.fdtd_pv_last_error.restype = ctypes.c_char_p
    return L


def _ptr(a):
    return ctypes.c_void_p(a.ctypes.data)


def _aligned(nbytes):
    a = np.zeros(nbytes + 256, np.uint8)
    off = (-a.ctypes.data) % 256
    return a[off:off + nbytes]


class Ctx:
    """One second-order context on host memory; shots: (n, cpml) each."""

    def __init__(self, L, shots, variant=0, storage=0, nt=64, nrec=5, less=0):
        self.L, self.keep = L, []
        arr = (_lib.ShotConfig * len(shots))()
        for s, (n, cpml) in zip(arr, shots):
            s.n[:], s.h[:], s.cpml[:] = n, (10.0,) * 3, cpml
            s.dt, s.exchange_every, s.R, s.kappa_max, s.alpha_frac = 1e-4, 1, 1e-8, 5.0, 0.05
            s.storage, s.variant, s.tblock_k, s.field_scale = storage, variant, 1, 1024.0 if storage else 0.0
        self.c = ctypes.c_void_p()
        assert L.fdtd_create(arr, len(shots), None, ctypes.byref(self.c)) == 0
        nb = ctypes.c_size_t()
        assert L.fdtd_workspace_size(self.c, ctypes.byref(nb)) == 0
        self.size = nb.value
        self.ws = _aligned(self.size)
        self.bound = L.fdtd_bind_workspace(self.c, _ptr(self.ws), ctypes.c_size_t(self.size - less))
        if self.bound != 0:
            return
        for i, (n, _) in enumerate(shots):
            self.model(i, n)
            self.source(i, (4, 4, 4), nt)
            rec, tr = self.hold(np.full((nrec, 3), 5, np.int32)), self.hold(np.zeros((nt, nrec), np.float32))
            assert L.fdtd_set_receivers(self.c, i, _ptr(rec), nrec) == 0
            assert L.fdtd_record_receivers(self.c, i, _ptr(tr), nt) == 0

    def hold(self, a):
        self.keep.append(a)
        return a

    def model(self, i, n):
        v = self.hold(np.full(n[::-1], 2000.0, np.float32))
        assert self.L.fdtd_set_velocity(self.c, i, _ptr(v)) == 0

    def source(self, i, at, nt=64):
        w = self.hold(np.ones(nt, np.float32))
        assert self.L.fdtd_inject_source(self.c, i, *at, _ptr(w), nt, ctypes.c_float(1.0)) == 0

    def close(self):
        self.L.fdtd_destroy(self.c)


@pytest.mark.parametrize("shots", [[((40, 36, 33), (8,) * 6)], [((40, 36, 33), (8,) * 6), ((33, 40, 36), (6,) * 6)]],
                         ids=["one", "two"])
def test_graph_kept_over_a_new_source_and_model(host, shots):
    """The captured steps read source and model from the device: a survey's loop of new source or model, reset and
    step as a graph captures once."""
    p = Ctx(host, shots)
    assert p.bound == 0
    host.stub_reset()
    for k in range(4):
        for i, (n, _) in enumerate(shots):
            p.source(i, (5 + k, 6, 7))
            p.model(i, n)
        assert host.fdtd_reset(p.c) == 0
        assert host.fdtd_step_graph(p.c, 10) == 0
    assert host.stub_instantiated() == 1
    assert host.stub_launches(b"k_tile") == 10      # (captured once, by the tile kernel)
    p.close()


class PV:
    """One first-order context on host memory."""

    def __init__(self, L, n, cpml=(5,) * 6, variant=0, less=0):
        self.L = L
        cfg = _lib.PVConfig()
        cfg.n[:], cfg.cpml[:], cfg.lam, cfg.variant = n, cpml, 0.05, variant
        self.c, self.stream = ctypes.c_void_p(), np.zeros(8, np.uint8)
        assert L.fdtd_pv_create(ctypes.byref(cfg), _ptr(self.stream), ctypes.byref(self.c)) == 0
        nb = ctypes.c_size_t()
        assert L.fdtd_pv_workspace_size(self.c, ctypes.byref(nb)) == 0
        self.size = nb.value
        self.ws = _aligned(self.size)
        self.bound = L.fdtd_pv_bind_workspace(self.c, _ptr(self.ws), ctypes.c_size_t(self.size - less))

    def steps(self, k):
        """(launches of the one-launch step, launches of the stages) of k steps."""
        self.L.stub_reset()
        assert self.L.fdtd_pv_step(self.c, k) == 0
        return tuple(self.L.stub_launches(name) for name in (b"k_pv_tile", b"k_pv_vel"))

    def close(self):
        self.L.fdtd_pv_destroy(self.c)


def test_captured_first_order_steps_end_in_the_buffers_they_began_in(host):
    """The one-launch step alternates between two buffers; a captured call, and every call after it, must not leave the
    state in the other one, where a replay would not find it."""
    p = PV(host, (40, 30, 20))
    assert p.bound == 0
    assert p.steps(3) == (3, 0)
    host.stub_capturing(1)
    try:
        assert p.steps(3) == (2, 1)
        assert p.steps(1) == (0, 1)
        assert p.steps(4) == (4, 0)
    finally:
        host.stub_capturing(0)
    assert p.steps(1) == (0, 1)
    assert p.steps(6) == (6, 0)
    p.close()


def test_first_order_workspace_of_ten_fields(host):
    """What holds the ten fields of the stages is accepted and stepped by them; one byte less is refused."""
    n = (40, 30, 20)
    least = PV(host, n, variant=1)
    p = PV(host, n)
    assert p.bound == 0 and p.steps(2) == (2, 0) and p.size > least.size
    gap = p.size - least.size
    q = PV(host, n, less=gap)
    assert q.bound == 0 and q.steps(2) == (0, 2)
    r = PV(host, n, less=gap + 1)
    assert r.bound == -4
    for c in (least, p, q, r):
        c.close()


@pytest.mark.parametrize("shots,variant", [([((40, 36, 33), (8,) * 6)], 1),
                                           ([((40, 36, 33), (8,) * 6), ((33, 40, 36), (6,) * 6)], 2)], ids=["one", "two"])
@pytest.mark.parametrize("storage", [0, 1])
def test_workspace_without_second_psi(host, shots, variant, storage):
    """What holds the shots of the explicit variant is accepted for the automatic one and stepped by its kernels; one
    byte less is refused, and the full size still takes the one launch."""
    least = Ctx(host, shots, variant, storage)
    p = Ctx(host, shots, 0, storage)
    gap = p.size - least.size
    assert p.bound == 0 and gap > 0
    q = Ctx(host, shots, 0, storage, less=gap)
    assert q.bound == 0
    for c, tiled in ((least, 0), (p, 4), (q, 0)):
        host.stub_reset()
        assert host.fdtd_step(c.c, 4) == 0
        assert host.stub_launches(b"k_tile") == tiled
    r = Ctx(host, shots, 0, storage, less=gap + 1)
    assert r.bound == -4
    assert host.fdtd_bind_workspace(r.c, _ptr(r.ws), ctypes.c_size_t(r.size)) == 0
    nb = ctypes.c_size_t()
    assert host.fdtd_workspace_size(r.c, ctypes.byref(nb)) == 0 and nb.value == p.size
    for c in (least, p, q, r):
        c.close()


# points at which a launch of its own for the interior begins: 1.2e7 in FP32, 1.6e7 in 16-bit storage (and k_face with it)
@pytest.mark.parametrize("shots,storage,launches", [
    ([((261, 243, 197), (10, 12, 9, 20, 15, 11))], 0, (1, 0, 1)),
    ([((256, 240, 200), (0, 20, 20, 0, 0, 20))], 0, (1, 0, 1)),
    ([((97, 200, 640), (20, 20, 90, 90, 20, 20))], 0, (1, 0, 1)),
    ([((261, 243, 197), (10, 12, 9, 20, 15, 11))], 1, (0, 0, 1)),
    ([((250, 240, 199), (20,) * 6)], 0, (0, 0, 1)),
    ([((283, 243, 237), (10, 12, 9, 20, 15, 11))], 1, (1, 1, 1)),
    ([((160, 170, 640), (20, 20, 70, 70, 20, 20))], 2, (1, 1, 1)),
    ([((129, 250, 512), (20, 2, 20, 20, 20, 20))], 2, (0, 1, 1)),     # no box fits between the x bands
    ([((180, 190, 200), (15,) * 6), ((200, 170, 180), (15, 10, 0, 9, 20, 15))], 0, (1, 0, 1)),
    ([((220, 190, 200), (15,) * 6), ((240, 200, 180), (15, 10, 0, 9, 20, 15))], 1, (1, 1, 1)),
    ([((220, 190, 200), (15,) * 6), ((240, 200, 180), (15, 10, 0, 9, 20, 15))], 2, (1, 1, 1)),
])
def test_launches_of_a_step(host, shots, storage, launches):
    """Which of k_inner, k_face and k_tile a step of these shots takes: the grids whose bits the GPU tests compare are
    those that reach the launches."""
    p = Ctx(host, shots, storage=storage)
    assert p.bound == 0
    host.stub_reset()
    assert host.fdtd_step(p.c, 1) == 0
    assert tuple(host.stub_launches(k) for k in (b"k_inner", b"k_face", b"k_tile")) == launches
    assert all(host.stub_blocks(k) > 0 for k, n in zip((b"k_inner", b"k_face", b"k_tile"), launches) if n)
    p.close()
