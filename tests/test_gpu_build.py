"""The corner table, edge numbering and lists of the feature build at the sizes where
their tiles, buckets and fan paths change, through the band they lead to, against the
oracle (agreement rules of parity.py); and the radix-sort path of the largest meshes
against a torus's closed form."""
import numpy as np
import pytest

import meshgen
import oracle
from meshgen import Grid
from parity import assert_parity, compare

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1903_00353_amd as P  # noqa: E402


def check(v, f, g):
    verts, tris = torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda()
    feats = P.csc_build_features(verts, tris, g)
    info = feats.info()
    assert info["n_edges"] == 3 * f.shape[0] // 2
    band = P.csc_scan_convert(feats)
    om = oracle.OracleMesh(v, f)
    rep = compare(om, g, om.band(g), band.cell.cpu().numpy(), band.sdf.cpu().numpy(), band.feat.cpu().numpy())
    print(rep, flush=True)
    assert rep["n_oracle"] > 0
    assert_parity(rep)


# faces at, below and above tiles of 256; vertices at the edges of the buckets' sizes
# (512 * 64 = 32768 with the vertices below)
@pytest.mark.parametrize("nu,nv", [(3, 3), (8, 16), (43, 3), (64, 64), (181, 179), (183, 180)])
def test_tiles_and_buckets(nu, nv):
    """A noisy torus with its vertices renumbered at random and vertices of no triangle
    before and after them (buckets without corners)."""
    rng = np.random.default_rng(1000 * nu + nv)
    v, f = meshgen.torus(nu, nv, noise=0.002, seed=nu)
    lone = rng.random((200, 3)).astype(np.float32)
    order = rng.permutation(v.shape[0])
    where = np.empty_like(order)
    where[order] = np.arange(order.size)
    v2 = np.ascontiguousarray(np.concatenate([lone[:70], v[order], lone[70:]]), dtype=np.float32)
    f2 = np.ascontiguousarray(where[f] + 70, dtype=np.int32)
    print("[case] build torus", nu, nv, "V", v2.shape[0], "F", f2.shape[0], flush=True)
    check(v2, f2, Grid.unit(32, 3))


@pytest.mark.parametrize("n", [3, 6, 7, 12, 13, 40])
def test_fan_degrees(n):
    """Apexes of degree n: the six corners sorted in registers, the ones inserted after
    them, the fans staged in LDS and those that are not."""
    v, f = meshgen.bipyramid(n)
    f = np.ascontiguousarray(f[np.random.default_rng(n).permutation(f.shape[0])])
    print("[case] build bipyramid", n, flush=True)
    check(v, f, Grid.unit(40, 3))


def test_more_vertices_than_the_buckets_hold():
    """16.8M vertices (over 2048 buckets of 8192): the corners are sorted by the radix
    sort. A torus of triangles far below a cell lies within 1e-6 of the exact torus;
    |SDF - closed form| stays within that and the FP32 tolerance of the distance."""
    nu, nv, N = 4096, 4104, 96
    R, r = 0.3, 0.12
    th = 2 * np.pi * torch.arange(nu, dtype=torch.float64, device="cuda").repeat_interleave(nv) / nu
    ph = 2 * np.pi * torch.arange(nv, dtype=torch.float64, device="cuda").repeat(nu) / nv
    w = R + r * ph.cos()
    verts = torch.stack([0.5 + w * th.cos(), 0.5 + w * th.sin(), 0.5 + r * ph.sin()], 1).float().contiguous()
    i = torch.arange(nu, device="cuda").repeat_interleave(nv)
    j = torch.arange(nv, device="cuda").repeat(nu)
    ip, jp = (i + 1) % nu, (j + 1) % nv
    a, b, c, d = i * nv + j, ip * nv + j, ip * nv + jp, i * nv + jp
    tris = torch.cat([torch.stack([a, b, c], 1), torch.stack([a, c, d], 1)]).int().contiguous()
    del th, ph, w, i, j, ip, jp, a, b, c, d
    g = Grid.unit(N, 3)
    print("[case] build torus of", verts.shape[0], "vertices", flush=True)
    feats = P.csc_build_features(verts, tris, g)
    assert feats.info()["n_edges"] == 3 * nu * nv
    band = P.csc_scan_convert(feats)
    cell = band.cell.long()
    x, y, z = ((q.double() + 0.5) / N - 0.5 for q in (cell % N, cell // N % N, cell // (N * N)))
    exact = torch.sqrt((torch.sqrt(x * x + y * y) - R) ** 2 + z * z) - r
    err = (band.sdf.double() - exact).abs().max().item()
    print("max error", err, flush=True)
    # the shell of half-width 3 h around the torus holds 2 * 3 h * 4 pi^2 R r in volume
    shell = 6.0 * 4.0 * np.pi ** 2 * R * r * N * N
    assert abs(band.n_band - shell) <= 0.01 * shell and err <= 1e-6 + 1e-5 / N


def test_band_offsets_at_the_store_sizes_of_both_scans():
    """The band's place in the outputs from the one-block scan of the bricks' counts, at
    the edges of its runs of 4096 and its largest store, against the general scan: the
    same offsets and cells, bit for bit."""
    parts = [meshgen.icosphere(3), meshgen.torus(24, 18), meshgen.icosphere(1)]
    grids = [Grid.unit(40, 3), Grid.unit(208, 3), Grid.unit(24, 3)]
    verts = torch.from_numpy(np.concatenate([v for v, _ in parts])).cuda()
    tris = torch.from_numpy(np.concatenate([f for _, f in parts])).cuda()
    f = P.csc_build_features_batched(verts, tris, [v.shape[0] for v, _ in parts], [t.shape[0] for _, t in parts], grids)
    nb = int(f.info()["n_bricks"])
    assert nb < 4095

    def scan(n):
        print("[case] store of", n, "bricks", flush=True)
        nbytes, mx = P.csc_scan_convert_workspace_for(f, n)
        out = tuple(torch.full((mx,), -7, dtype=t, device="cuda") for t in (torch.float32, torch.int32, torch.int32))
        off = torch.full((len(parts) + 1,), -1, dtype=torch.int64, device="cuda")
        P.csc_scan_convert_batched(f, torch.empty(nbytes, dtype=torch.uint8, device="cuda"), out, off)
        off = off.cpu().tolist()
        return off, [o[:off[-1]].cpu() for o in out]

    off, out = scan(16385)  # the general scan
    assert off[0] == 0 and all(a < b for a, b in zip(off, off[1:]))
    for n in (nb, 4095, 4096, 4097, 8193, 16384):
        got_off, got = scan(n)
        assert got_off == off
        assert all(torch.equal(a, b) for a, b in zip(got, out))


def n_bricks(meshes, grids):
    verts = torch.from_numpy(np.concatenate([v for v, _ in meshes])).cuda()
    tris = torch.from_numpy(np.concatenate([f for _, f in meshes])).cuda()
    return int(P.csc_build_features_batched(verts, tris, [v.shape[0] for v, _ in meshes],
                                            [t.shape[0] for _, t in meshes], grids).info()["n_bricks"])


@pytest.mark.parametrize("mesh,grid", [(meshgen.icosphere(0), Grid.unit(100, 3)), (meshgen.icosphere(1), Grid.unit(70, 9)),
                                       (meshgen.icosphere(3), Grid.unit(33, 1.5)), (meshgen.torus(11, 6), Grid.unit(257, 2))])
def test_bricks_marked_by_the_block_and_by_the_thread(mesh, grid):
    """Few faces, whose bricks the block marks together, alone and behind so many faces
    that each thread marks its own: the same number of bricks."""
    many = meshgen.torus(300, 230)
    assert many[1].shape[0] > 1 << 17
    print("[case] bricks", mesh[1].shape, tuple(grid.n), flush=True)
    alone = n_bricks([mesh], [grid])
    assert alone > 0
    rest = n_bricks([many], [Grid.unit(32, 2)])
    assert n_bricks([many, mesh], [Grid.unit(32, 2), grid]) == rest + alone
    # two meshes of few faces: the descriptor is read per face
    assert n_bricks([mesh, meshgen.icosphere(2)], [grid, Grid.unit(24, 2)]) == \
        alone + n_bricks([meshgen.icosphere(2)], [Grid.unit(24, 2)])


@pytest.mark.parametrize("n", [3, 6, 7, 8, 9, 12, 13, 40])
def test_fans_by_lanes_and_by_threads(n):
    """A mesh of few vertices alone, its fans taken by lanes, and behind so many vertices
    that a thread takes each: the same band, bit for bit."""
    many = meshgen.torus(300, 230)
    v, f = meshgen.bipyramid(n)
    g = Grid.unit(40, 3)
    assert v.shape[0] <= 1 << 16 < many[0].shape[0]
    print("[case] fans", n, flush=True)
    alone, behind = P.Batch([(v, f)], [g]), P.Batch([many, (v, f)], [Grid.unit(32, 2), g])
    for b in (alone, behind):
        b.step()
        b.check()
    got, want = alone.band(0), behind.band(1)
    assert want[0].numel() > 0
    assert all(torch.equal(x, y) for x, y in zip(got, want))
