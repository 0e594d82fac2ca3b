"""The adjoint's table of vertices where it is crowded: more vertices met by a block's
chunk of cells than its slots hold, next to chunks that meet few, against the oracle."""
import numpy as np
import pytest

import meshgen
import oracle
from meshgen import Grid
from parity import assert_same_sums, vertex_term_scale

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1903_00353_amd as P  # noqa: E402


@pytest.mark.parametrize("far", [False, True])
def test_crowded_table(far):
    """A fine sphere (several vertices per cell of its surface) alone, every chunk
    crowded; and with a coarse tetrahedron-like bipyramid before it in a batch, so that
    runs of cells go from large faces to small ones. Every vertex within 1e-5 of the sum of
    the magnitudes of its terms (the rule of the other adjoint tests)."""
    meshes, grids = [meshgen.icosphere(8)], [Grid.unit(400, 1.5)]
    if far:
        meshes, grids = [meshgen.bipyramid(5), meshes[0]], [Grid.unit(150, 6), grids[0]]
    print("[case] crowded table", far, flush=True)
    B = P.Batch(meshes, grids)
    B.step()
    B.check()
    off = B.band_off.cpu().tolist()
    assert off[-1] > 2048 * 256  # two chunks of cells and more for some block
    for m, ((v, f), g) in enumerate(zip(meshes, grids)):
        sdf, feat, cell = (x.cpu().numpy() for x in B.band(m))
        om = oracle.OracleMesh(v, f)
        up = 2.0 * sdf.astype(np.float64)
        ref = om.grad(g, cell, feat, np.sign(sdf), up)
        assert_same_sums(B.grad(m).cpu().numpy(), ref, vertex_term_scale(f, om.edges, v.shape[0], feat, up), m)
