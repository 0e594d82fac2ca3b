"""Handles made and freed one after another and from several threads: the device memory
that one leaves serves the next, with results as of a handle kept from the start."""
import threading

import numpy as np
import pytest

import meshgen
from meshgen import Grid

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1903_00353_amd as P  # noqa: E402

CASES = [(meshgen.icosphere(2), Grid.unit(24, 3)), (meshgen.torus(40, 30), Grid.unit(64, 3)),
         (meshgen.icosphere(4), Grid.unit(40, 2)), (meshgen.torus(64, 48), Grid.unit(96, 4))]


def pass_of(case):
    """One build, scan and adjoint whose handle is freed with the adjoint still queued."""
    (v, t), g = case
    verts, tris = torch.from_numpy(v).cuda(), torch.from_numpy(t).cuda()
    f = P.csc_build_features(verts, tris, g)
    band = P.csc_scan_convert(f)
    grad = P.csc_sdf_backward(f, band, torch.ones_like(band.sdf))
    f.free()
    return band.sdf, band.feat, band.cell, grad


def agree(got, want):
    for a, b in zip(got[:3], want[:3]):
        assert torch.equal(a, b)
    # sums of atomically added floats: the order of the additions may differ
    assert torch.allclose(got[3], want[3], rtol=0, atol=1e-5 * float(want[3].abs().max()) + 1e-6)


def test_handles_one_after_another():
    want = [pass_of(c) for c in CASES]
    torch.cuda.synchronize()
    rng = np.random.default_rng(5)
    for k in rng.integers(len(CASES), size=24):
        print("[case] pass", k, flush=True)
        agree(pass_of(CASES[k]), want[k])


def test_handles_of_threads_on_their_own_streams():
    want = [pass_of(c) for c in CASES]
    torch.cuda.synchronize()
    errors = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(10):
                    got = pass_of(CASES[(k + i) % len(CASES)])
                    torch.cuda.current_stream().synchronize()
                    agree(got, want[(k + i) % len(CASES)])
        except BaseException as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    print("[case] four threads", flush=True)
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_kept_memory_is_bounded():
    """Many handles alive at once, then freed: no more than the documented 256 MiB (and the
    allocator's own rounding of 2 MiB for each kept block) stays."""
    v, t = meshgen.icosphere(6)
    verts, tris = torch.from_numpy(v).cuda(), torch.from_numpy(t).cuda()
    P.csc_build_features(verts, tris, Grid.unit(128, 3)).free()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    print("[case] thirty handles", flush=True)
    handles = [P.csc_build_features(verts, tris, Grid.unit(128, 3)) for _ in range(30)]
    assert before - torch.cuda.mem_get_info()[0] > (400 << 20)
    for h in handles:
        h.free()
    assert before - torch.cuda.mem_get_info()[0] <= (256 + 16 * 2) << 20
