"""What the library's host code keeps and gives back, without a GPU: its objects linked
against a stand-in for the HIP runtime (host_runtime.cpp), which runs no kernel."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

import paper_1903_00353_amd as P
from paper_1903_00353_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
OBJECTS = os.path.join(build.OUT_DIR, "obj")
OK, OUT_OF_MEMORY, HIP_ERROR = 0, 6, 7


class Sim:
    """The library on the stand-in, in its initial state."""

    def __init__(self, path):
        self.lib = C.CDLL(path)
        self.lib.csc_build_features_batched.argtypes = P.lib().csc_build_features_batched.argtypes
        self.lib.csc_features_order_faces.argtypes = [C.c_void_p, C.c_int32, C.c_void_p]
        self.lib.csc_features_free.argtypes = [C.c_void_p]
        self.lib.csc_weld_soup.argtypes = P.lib().csc_weld_soup.argtypes

    def __getattr__(self, name):  # a variable of the stand-in
        return (C.c_size_t if name in ("limit", "used") else C.c_int).in_dll(self.lib, "sim_" + name)

    def build(self, n, out=None, meshes=5, nv=6, nf=8, stream=None):
        """(status, handle) of `meshes` equal meshes on grids of n^3 cells; five meshes
        have their tables copied, four or fewer as kernel arguments."""
        out = C.c_void_p() if out is None else out
        grids = (P.csc_grid * meshes)()
        for g in grids:
            g.n[:] = [n, n, n]
            g.h, g.band_cells = 1.0 / n, 2.0
        data = C.c_void_p(0x1000)  # handed to kernels only
        code = self.lib.csc_build_features_batched(data, data, (C.c_int64 * meshes)(*[nv] * meshes),
                                                   (C.c_int64 * meshes)(*[nf] * meshes), grids, meshes, None, 0, stream,
                                                   C.byref(out))
        return code, out


@pytest.fixture
def sim(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    objects = [os.path.join(OBJECTS, os.path.splitext(s)[0] + ".o") for s in build.SOURCES]
    if not all(os.path.exists(o) for o in objects):
        build.build()
    include = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc()))), "include")
    path = str(tmp_path / "libsim.so")
    subprocess.run([cxx, "-std=c++17", "-shared", "-fPIC", "-I" + include, os.path.join(HERE, "host_runtime.cpp"),
                    *objects, "-Wl,-Bsymbolic", "-lpthread", "-o", path], check=True)
    return Sim(path)


def test_a_build_refused_under_capture_leaves_the_tables_of_the_one_before(sim):
    """A changed configuration is refused while its stream is captured; the next build with
    the former one finds its tables in the memory that it uses."""
    code, h = sim.build(16)
    assert code == OK and sim.uploads.value == 4
    sim.capturing.value = 1
    assert sim.build(160, h)[0] == HIP_ERROR
    sim.capturing.value = 0
    assert sim.build(16, h)[0] == OK
    assert sim.uploads.value >= 4  # none since the last allocation: tables never written there
    # and a configuration that is accepted writes its own
    before = sim.uploads.value
    assert sim.build(24, h)[0] == OK and sim.uploads.value == before + 4
    sim.lib.csc_features_free(h)


def test_a_build_that_runs_out_of_memory_writes_its_tables_the_next_time(sim):
    code, h = sim.build(16)
    assert code == OK
    sim.limit.value = sim.used.value
    assert sim.build(160, h)[0] == OUT_OF_MEMORY
    sim.limit.value = 1 << 40
    assert sim.build(16, h)[0] == OK
    assert sim.uploads.value >= 4
    sim.lib.csc_features_free(h)


@pytest.mark.parametrize("stream", [None, 0x10])
def test_a_handle_freed_during_a_capture_is_waited_for_without_ending_it(sim, stream):
    """hipDeviceSynchronize would end the capture (of any thread); hipFree, which waits for
    the device too, is called where the handle was used on another than the null stream.
    The handle's memory serves the next one all the same."""
    code, h = sim.build(16, stream=stream)
    assert code == OK
    frees = sim.frees.value
    sim.capturing.value = 1
    sim.lib.csc_features_free(h)
    sim.capturing.value = 0
    assert sim.device_waits.value == 0
    assert (sim.frees.value > frees) == (stream is not None)
    used = sim.used.value
    code, h = sim.build(16)
    assert code == OK and sim.used.value == used
    sim.lib.csc_features_free(h)


def test_kept_memory_serves_every_allocation_that_runs_out(sim):
    """With no room left but what a freed handle's memory takes, the face order gets its
    memory all the same."""
    code, h = sim.build(16)
    code2, kept = sim.build(64)
    assert code == OK and code2 == OK
    sim.lib.csc_features_free(kept)
    sim.limit.value = sim.used.value
    assert sim.lib.csc_features_order_faces(h, 1, None) == OK
    sim.lib.csc_features_free(h)


def test_a_face_order_is_refused_under_capture(sim):
    """Before anything is allocated, freed or queued."""
    code, h = sim.build(16)
    assert code == OK
    allocs, frees = sim.allocs.value, sim.frees.value
    sim.capturing.value = 1
    assert sim.lib.csc_features_order_faces(h, 1, 0x10) == HIP_ERROR
    sim.capturing.value = 0
    assert (sim.allocs.value, sim.frees.value) == (allocs, frees)
    assert sim.lib.csc_features_order_faces(h, 1, None) == OK
    sim.lib.csc_features_free(h)


def test_kept_memory_is_given_back_on_request(sim):
    handles = [sim.build(n, stream=s)[1] for n in (16, 64) for s in (None, 0x10)]
    live, h = sim.used.value, handles.pop()
    for x in handles:
        sim.lib.csc_features_free(x)
    assert live // 2 < sim.used.value <= live + 64  # kept (and the one small allocation)
    sim.lib.csc_release_memory()
    one = sim.used.value
    assert 0 < one < live // 2  # what the handle in use takes
    sim.lib.csc_features_free(h)
    sim.lib.csc_release_memory()
    assert sim.used.value <= 64


def test_a_weld_is_refused_under_capture(sim):
    """Before it takes scratch memory, whose free could fail there."""
    data, nv = C.c_void_p(0x1000), C.c_int64()
    sim.capturing.value = 1
    assert sim.lib.csc_weld_soup(data, 1 << 16, data, data, C.byref(nv), 0x10) == HIP_ERROR
    sim.capturing.value = 0
    assert sim.allocs.value == 0 and sim.used.value == 0
    assert sim.lib.csc_weld_soup(data, 1 << 16, data, data, C.byref(nv), 0x10) == OK


@pytest.mark.parametrize("nf,ordered", [(1 << 16, False), (7 << 20, True)])
def test_scratch_too_large_to_keep_is_allocated_in_stream_order(sim, nf, ordered):
    """The scratch of a weld of 7.3M faces passes 256 MiB: it is not freed by hipFree, which
    would wait for the work of other streams. A smaller one is kept."""
    data, nv = C.c_void_p(0x1000), C.c_int64()
    for _ in range(2):
        assert sim.lib.csc_weld_soup(data, nf, data, data, C.byref(nv), None) == OK
    assert sim.ordered_allocs.value == (2 if ordered else 0) and sim.frees.value == 0
    assert sim.allocs.value == (2 if ordered else 1)
    assert (sim.used.value == 0) == ordered
