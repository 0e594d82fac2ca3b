"""Handles while a graph is being captured: what is refused there and what is not."""
import threading

import pytest

import meshgen
from meshgen import Grid

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1903_00353_amd as P  # noqa: E402


def mesh(level):
    v, t = meshgen.icosphere(level)
    return torch.from_numpy(v).cuda(), torch.from_numpy(t).cuda()


@pytest.mark.parametrize("meshes", [1, 5])
def test_a_changed_configuration_is_refused_under_capture(meshes):
    """The handle is then rebuilt with its former configuration and gives that field, and
    the capture that met the refusal ends well. One mesh's tables travel as kernel
    arguments, those of five are copied."""
    v, t = mesh(3)
    nv, nf = v.shape[0], t.shape[0]
    verts, tris = v.repeat(meshes, 1).contiguous(), t.repeat(meshes, 1).contiguous()
    x = torch.ones(100, device="cuda")

    def build(n, reuse=None):
        return P.csc_build_features_batched(verts, tris, [nv] * meshes, [nf] * meshes, [Grid.unit(n, 3)] * meshes,
                                            reuse=reuse)

    f, kept = build(32), build(32)
    torch.cuda.synchronize()
    print("[case] refused under capture", meshes, flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = x * 2
        with pytest.raises(P.CscError):
            build(160, reuse=f)
        z = y + 1
    g.replay()
    assert z[0].item() == 3.0
    build(32, reuse=f)

    def scan(h):
        nbytes, mx = P.csc_scan_convert_workspace(h)
        out = tuple(torch.zeros(mx, dtype=d, device="cuda") for d in (torch.float32, torch.int32, torch.int32))
        off = torch.zeros(meshes + 1, dtype=torch.int64, device="cuda")
        P.csc_scan_convert_batched(h, torch.empty(nbytes, dtype=torch.uint8, device="cuda"), out, off)
        return (off,) + out

    assert f.info() == kept.info()
    assert all(torch.equal(a, b) for a, b in zip(scan(f), scan(kept)))


def test_calls_refused_under_capture_leave_it_alone():
    """A weld, which synchronises, and a face order: refused, and the capture goes on."""
    verts, tris = mesh(3)
    f = P.csc_build_features(verts, tris, Grid.unit(32, 3))
    soup = verts[tris.long()].contiguous()
    P.csc_weld_soup(soup)
    x = torch.ones(100, device="cuda")
    torch.cuda.synchronize()
    print("[case] refused calls", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = x * 2
        for call in (lambda: P.csc_features_order_faces(f), lambda: P.csc_weld_soup(soup)):
            with pytest.raises(P.CscError) as e:
                call()
            assert e.value.code == 7
        z = y + 1
    g.replay()
    assert z[0].item() == 3.0
    P.csc_features_order_faces(f)
    assert P.csc_weld_soup(soup)[0].shape == verts.shape


@pytest.mark.parametrize("thread", [False, True])
@pytest.mark.parametrize("mode", ["relaxed", "thread_local", "global"])
def test_a_handle_is_freed_during_a_capture(mode, thread):
    """By the capturing thread or by another: the capture ends well, and a handle that
    takes the memory over gives its field."""
    verts, tris = mesh(3)
    f = P.csc_build_features(verts, tris, Grid.unit(32, 3))
    want = P.csc_scan_convert(f)
    x = torch.ones(100, device="cuda")
    torch.cuda.synchronize()
    print("[case] free during capture", mode, thread, flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode=mode):
        y = x * 2
        if thread:
            t = threading.Thread(target=f.free)
            t.start()
            t.join()
        else:
            f.free()
        z = y + 1
    for _ in range(3):
        z.zero_()
        g.replay()
        assert z[0].item() == 3.0
    got = P.csc_scan_convert(P.csc_build_features(verts, tris, Grid.unit(32, 3)))
    assert all(torch.equal(a, b) for a, b in zip((got.sdf, got.feat, got.cell), (want.sdf, want.feat, want.cell)))


@pytest.mark.parametrize("level,n", [(3, 48), (5, 440)])  # one-block and general scan of the store's counts
def test_a_workspace_on_an_8_byte_boundary(level, n):
    """The keys are 8 bytes wide and need no more: the same field as from the allocator's
    own boundary."""
    verts, tris = mesh(level)
    f = P.csc_build_features(verts, tris, Grid.unit(n, 12))
    nbytes, _ = P.csc_scan_convert_workspace(f)
    print("[case] workspace at 8 bytes", level, n, flush=True)
    want = P.csc_scan_convert(f, torch.full((nbytes,), 1, dtype=torch.uint8, device="cuda"))
    got = P.csc_scan_convert(f, torch.full((nbytes + 8,), 1, dtype=torch.uint8, device="cuda")[8:])
    assert want.n_band > 0
    assert all(torch.equal(a, b) for a, b in zip((got.sdf, got.feat, got.cell), (want.sdf, want.feat, want.cell)))


def test_a_handle_freed_with_work_on_another_stream():
    """Built on one stream, scanned on another behind some milliseconds of other work, then
    freed: its memory serves the next handle only once that scan is done."""
    verts, tris = mesh(4)
    g = Grid.unit(64, 3)
    want = P.csc_scan_convert(P.csc_build_features(verts, tris, g))
    other = P.csc_build_features(verts * 0.5, tris, g)
    other.free()
    side = torch.cuda.Stream()
    a = torch.rand(4096, 4096, device="cuda")
    f = P.csc_build_features(verts, tris, g)
    nbytes, mx = P.csc_scan_convert_workspace(f)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    out = (torch.zeros(mx, device="cuda"), torch.zeros(mx, dtype=torch.int32, device="cuda"),
           torch.zeros(mx, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda"))
    torch.cuda.synchronize()
    print("[case] freed behind another stream", flush=True)
    with torch.cuda.stream(side):
        for _ in range(10):
            b = a @ a
        P.csc_scan_convert(f, ws, out, sync_count=False)
    f.free()
    P.csc_build_features(verts * 0.5, tris, g)  # takes the memory over
    torch.cuda.synchronize()
    assert b.shape == a.shape and int(out[3].item()) == want.n_band
    assert all(torch.equal(x[:want.n_band], y) for x, y in zip(out, (want.sdf, want.feat, want.cell)))


def test_kept_memory_is_given_back_on_request():
    v, t = meshgen.icosphere(7)
    verts, tris = torch.from_numpy(v).cuda(), torch.from_numpy(t).cuda()
    f = P.csc_build_features(verts, tris, Grid.unit(64, 3))
    P.csc_release_memory()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    print("[case] release", flush=True)
    f.free()
    assert torch.cuda.mem_get_info()[0] - free < 4 << 20  # kept
    P.csc_release_memory()
    assert torch.cuda.mem_get_info()[0] - free > 64 << 20  # the arena of 328,000 faces
    got = P.csc_scan_convert(P.csc_build_features(verts, tris, Grid.unit(64, 3)))
    assert got.n_band > 0


@pytest.mark.parametrize("nu,nv", [(400, 300), (2048, 1600)])  # scratch kept; above 256 MiB
def test_a_weld_waits_for_no_other_stream(nu, nv):
    i = torch.arange(nu, device="cuda").repeat_interleave(nv)
    j = torch.arange(nv, device="cuda").repeat(nu)
    ip, jp = (i + 1) % nu, (j + 1) % nv
    a, b, c, d = i * nv + j, ip * nv + j, ip * nv + jp, i * nv + jp
    tris = torch.cat([torch.stack([a, b, c], 1), torch.stack([a, c, d], 1)])
    pos = torch.stack([torch.arange(nu * nv, device="cuda") % 4096, torch.arange(nu * nv, device="cuda") // 4096,
                       torch.zeros(nu * nv, device="cuda", dtype=torch.long)], 1).float()
    soup = pos[tris].contiguous()
    del i, j, ip, jp, a, b, c, d
    P.csc_weld_soup(soup)  # the binding's outputs are in the allocator's cache from here on
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    m = torch.rand(8192, 8192, device="cuda")
    out = torch.empty_like(m)
    with torch.cuda.stream(side):
        torch.mm(m, m, out=out)  # the library is loaded
    torch.cuda.synchronize()
    print("[case] weld beside another stream", tris.shape[0], flush=True)
    with torch.cuda.stream(side):
        for _ in range(40):  # some 300 ms
            torch.mm(m, m, out=out)
        done.record()
    verts, got = P.csc_weld_soup(soup)
    waited = done.query()
    torch.cuda.synchronize()
    assert verts.shape[0] == nu * nv and torch.equal(verts[got.long()], soup)
    assert not waited
