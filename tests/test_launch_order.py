"""Calls of one context on different streams wait for each other: the library's host code linked with
a record of its HIP calls (order_recorder.cpp) in place of the runtime and the kernels, no GPU."""
import ctypes as C
import itertools
import os
import subprocess

import numpy as np
import pytest

from paper_1504_06570_amd import phx
from paper_1504_06570_amd.scene import coatings
from paper_1504_06570_amd.scene import configs
from paper_1504_06570_amd.scene.physics import tma_extras
from paper_1504_06570_amd.scene.readout import Readout

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Recorded:
    """A context of the recorded library with a coated telescope and three sources."""

    def __init__(self, path, monkeypatch):
        monkeypatch.setattr(phx, "LIB_PATH", str(path))
        monkeypatch.setattr(phx, "_lib", None)
        self.L = phx.lib()
        self.L.rec_overlaps.restype = C.c_char_p
        self.L.rec_capture.argtypes = [C.c_void_p, C.c_int]
        self.scene = configs.telescope(scale=1e-5)
        h = C.c_void_p()
        self.L.phx_create(0, C.byref(h))
        self.ctx = h
        self.load_prescription()
        t = np.ascontiguousarray(self.scene.coatings, np.float32)
        self.check(self.L.phx_load_coatings(h, t.ctypes.data, *t.shape, coatings.S_MAX, coatings.LAM0,
                                            coatings.DLAM))
        self.load_sources()
        self.memory = np.zeros(1 << 16)          # any output buffer: nothing writes to it
        self.image = np.zeros((128, 128), np.uint32)
        self.readout = phx.readout_struct(Readout(amp_nx=2, amp_ny=2))
        self.adu = np.zeros(1 << 16, np.uint16)
        self.L.rec_reset()

    def check(self, rc):
        assert rc == 0, self.L.phx_last_error(self.ctx)

    def load_prescription(self):
        self.check(self.L.phx_load_prescription(
            self.ctx, C.byref(phx.prescription_struct(self.scene.prescription))))

    def load_sources(self):
        self.scene.sources.n_photons[:] = 1000
        self.check(self.L.phx_load_sources(self.ctx, phx.sources_struct(self.scene.sources), 3, None,
                                           None, 0, 0))

    def load_reflectance(self):
        t = np.zeros_like(self.scene.coatings, np.float32)
        self.check(self.L.phx_load_reflectance(self.ctx, t.ctypes.data, *t.shape))

    def load_physics(self):
        self.check(self.L.phx_load_physics(self.ctx, C.byref(phx.physics_struct(tma_extras()))))

    def load_screens(self):
        a = phx.Atmosphere()
        a.n_layers, a.n_scales, a.screen_n, a.lambda_ref = 1, 1, 4, 500e-9
        a.height[0], a.pixel[0] = 1000.0, 1.0
        self.check(self.L.phx_load_screens(self.ctx, C.byref(a), self.memory.ctypes.data, 16, None))

    def perturb(self):
        th = (C.c_double * phx.N_THETA)(*([1e-5] * phx.N_THETA))
        self.check(self.L.phx_set_perturbation(self.ctx, th, phx.N_THETA))

    def args(self, photons):
        a = phx.TraceArgs()
        a.seed, a.flags, a.src_begin, a.src_end = 1, int(self.scene.physics) | phx.F_CULL, 0, 3
        a.photon_count = photons
        a.image_dev = self.memory.ctypes.data
        return a

    def call(self, name, stream, photons=1000):
        m, st = self.memory.ctypes.data, C.c_void_p(stream)
        if name in ("trace", "trace_batched", "trace_noalloc"):
            self.check(getattr(self.L, "phx_" + name)(self.ctx, C.byref(self.args(photons)), st))
        elif name == "adjoint":
            self.check(self.L.phx_adjoint(self.ctx, C.byref(self.args(photons)), m, m, None, 0, 0, st))
        elif name == "adjoint_moments":
            self.check(self.L.phx_adjoint_moments(self.ctx, C.byref(self.args(photons)), m, m, m, None,
                                                  0, 0, st))
        elif name == "readout":
            side = 64 if photons <= 1000 else 128
            self.check(self.L.phx_readout(self.ctx, C.byref(self.readout), self.image.ctypes.data, side,
                                          side, self.adu.ctypes.data, self.adu.size, None, None, None,
                                          st))

    def overlaps(self):
        return self.L.rec_overlaps().decode()


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    so = tmp_path_factory.mktemp("order") / "librecorded.so"
    subprocess.check_call(
        ["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__",
         "-I/opt/rocm/include", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", str(so),
         os.path.join(ROOT, "paper_1504_06570_amd", "csrc", "phx_api.cpp"),
         os.path.join(ROOT, "tests", "order_recorder.cpp")])
    return so


@pytest.fixture
def rec(library, monkeypatch):
    r = Recorded(library, monkeypatch)
    yield r
    r.L.phx_destroy(r.ctx)


CALLS = ["trace", "trace_batched", "adjoint", "adjoint_moments", "readout", "trace_noalloc"]


@pytest.mark.parametrize("first,second", list(itertools.product(CALLS, CALLS)))
def test_calls_on_two_streams_wait_for_each_other(rec, first, second):
    """Alternating streams, sizes that grow the workspaces and ones that reuse them, with the parameter
    block changed on the way: no operation starts before an earlier one is complete."""
    for photons in (1000, 1000, 100000, 1000):
        rec.call(first, 0x11, photons)
        rec.call(second, 0x22, photons)
        rec.perturb()
        rec.call(second, 0x11, photons)
    assert rec.overlaps() == ""
    assert rec.L.rec_operations() >= 12


def test_the_record_sees_a_missing_wait(rec, library, monkeypatch):
    """Two contexts do not order each other: the record says that their calls may overlap."""
    other = Recorded(library, monkeypatch)
    rec.call("trace", 0x11)
    assert rec.overlaps() == ""
    other.call("trace", 0x22)
    assert "may overlap trace" in rec.overlaps()
    other.L.phx_destroy(other.ctx)


@pytest.mark.parametrize("name", CALLS)
def test_a_captured_stream_gets_no_events(rec, name):
    rec.call(name, 0x11)
    rec.L.rec_reset()
    rec.L.rec_capture(0x22, 1)
    rec.call(name, 0x22)
    rec.L.rec_capture(0x22, 0)
    assert rec.L.rec_capture_events() == 0


def test_the_call_without_allocation_makes_nothing(rec):
    """phx_trace_noalloc as the context's first launch and after others: no memory, stream or event."""
    rec.call("trace_noalloc", 0x11)
    assert rec.L.rec_resources() == 0
    rec.call("trace", 0x22)
    before = rec.L.rec_resources()
    rec.call("trace_noalloc", 0x11, 100000)
    assert rec.L.rec_resources() == before and rec.overlaps() == ""


@pytest.mark.parametrize("load", ["reflectance", "physics", "screens", "prescription", "sources"])
def test_loads_wait_for_the_launch_that_reads_what_they_overwrite(rec, load):
    getattr(rec, "load_" + load)()
    rec.call("trace", 0x11)
    getattr(rec, "load_" + load)()          # tables of the same size
    rec.call("trace", 0x22)
    assert rec.overlaps() == ""
