"""Fans of more corners than a vertex has lanes, alone and among others in a wavefront:
the same field as from a thread per vertex, bit for bit, and the oracle's."""
import numpy as np
import pytest

import meshgen
import oracle
from meshgen import Grid
from parity import assert_parity, compare

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1903_00353_amd as P  # noqa: E402


def random_sphere(n, seed):
    """Delaunay triangles of n random points on a sphere: degrees 3 to 13."""
    hull = pytest.importorskip("scipy.spatial").ConvexHull
    rng = np.random.default_rng(seed)
    p = rng.normal(size=(n, 3))
    p /= np.linalg.norm(p, axis=1)[:, None]
    f = hull(p).simplices
    inward = np.einsum("ij,ij->i", np.cross(p[f[:, 1]] - p[f[:, 0]], p[f[:, 2]] - p[f[:, 0]]), p[f[:, 0]]) < 0
    f[inward] = f[inward][:, ::-1]
    return (0.5 + 0.35 * p).astype(np.float32), np.ascontiguousarray(f[rng.permutation(len(f))], dtype=np.int32)


def shuffled(mesh, seed):
    v, f = mesh
    return v, np.ascontiguousarray(f[np.random.default_rng(seed).permutation(f.shape[0])])


CASES = [("bipyramid %d" % n, shuffled(meshgen.bipyramid(n), n)) for n in (8, 9, 10, 15, 16, 17, 130)]


@pytest.mark.parametrize("name,mesh", CASES + [("random", None)], ids=[n for n, _ in CASES] + ["random"])
def test_fans_of_more_corners_than_lanes(name, mesh):
    v, f = mesh if mesh else random_sphere(3001, 7)
    if mesh is None:
        degree = np.bincount(f.ravel())
        assert degree.max() > 8 and degree.min() < 6
    g = Grid.unit(40, 3)
    many = meshgen.torus(300, 230)
    assert v.shape[0] <= 1 << 16 < many[0].shape[0]
    print("[case] fans", name, flush=True)
    alone, behind = P.Batch([(v, f)], [g]), P.Batch([many, (v, f)], [Grid.unit(32, 2), g])
    for b in (alone, behind):
        b.step()
        b.check()
    got, want = alone.band(0), behind.band(1)
    assert want[0].numel() > 0
    assert all(torch.equal(x, y) for x, y in zip(got, want))
    om = oracle.OracleMesh(v, f)
    rep = compare(om, g, om.band(g), got[2].cpu().numpy(), got[0].cpu().numpy(), got[1].cpu().numpy())
    print(rep, flush=True)
    assert_parity(rep)


@pytest.mark.parametrize("nu,nv", [(300, 230), (1200, 1180)])  # buckets of 256 and of 1024 threads
def test_fans_that_are_sorted_where_their_corners_are_placed(nu, nv):
    """Several long fans in one bucket, of fewer and more corners than a wavefront has lanes
    and of whole multiples: the same fields as each mesh gives alone."""
    many = meshgen.torus(nu, nv)
    parts = [shuffled(meshgen.bipyramid(n), n) for n in (13, 63, 64, 65, 100)]
    g = Grid.unit(40, 3)
    print("[case] long fans behind", many[1].shape[0], flush=True)
    behind = P.Batch([many] + parts, [Grid.unit(32, 2)] + [g] * len(parts))
    behind.step()
    behind.check()
    for k, part in enumerate(parts):
        alone = P.Batch([part], [g])
        alone.step()
        alone.check()
        got, want = behind.band(1 + k), alone.band(0)
        assert want[0].numel() > 0
        assert all(torch.equal(x, y) for x, y in zip(got, want))
