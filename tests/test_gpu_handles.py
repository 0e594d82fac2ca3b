"""Handles while a graph is being captured: what is refused there and what is not."""
import pytest

import meshgen
from meshgen import Grid

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1903_00353_amd as P  # noqa: E402


def mesh(level):
    v, t = meshgen.icosphere(level)
    return torch.from_numpy(v).cuda(), torch.from_numpy(t).cuda()


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip((a.sdf, a.feat, a.cell), (b.sdf, b.feat, b.cell)))


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
