"""The adjoint's block sums are exact also after a chunk of cells that crowds the table."""
import numpy as np
import pytest

import meshgen
from meshgen import Grid

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1903_00353_amd as P  # noqa: E402


def test_terms_that_cancel_after_a_crowded_chunk():
    """Every block takes two chunks of 256 cells. The first meets 256 faces (up to 768
    vertices, more than the table holds); in the second 85 vertices get the terms A, a
    and -A each, a about 2^-12 A, at the same cell. Summed exactly that is the term a, bit
    for bit what the band gives with A and -A left out; a term added to the gradient by
    itself would be rounded at A. (85 vertices in an emptied table of several hundred
    slots: all find a slot.)"""
    v, t = meshgen.icosphere(8)
    nv, nf = v.shape[0], t.shape[0]
    n = 64
    f = P.csc_build_features(torch.from_numpy(v).cuda(), torch.from_numpy(t).cuda(), Grid.unit(n, 2))
    blocks, rng = 2048, np.random.default_rng(3)
    used = rng.permutation(nv)[:85 * 512].reshape(512, 85)  # the vertices of blocks 0, 4, 8, ...
    mark = np.zeros(nv, bool)
    mark[used] = True
    other = np.flatnonzero(~mark[t].any(1))  # faces away from them
    feat = rng.choice(other, (blocks, 2, 256)).astype(np.int32)
    cell = rng.integers(n ** 3, size=(blocks, 2, 256), dtype=np.int32)
    up = np.full((blocks, 2, 256), 1000.0, np.float32)
    up[:, 1] = 0
    feat[::4, 1, :255] = np.tile(nf + 3 * nf // 2 + used, 3)
    cell[::4, 1, :255] = np.tile(cell[::4, 1, :85], 3)
    small = (0.25 * (1 + rng.random((512, 85)))).astype(np.float32)
    up[::4, 1, :255] = np.concatenate([np.full((512, 85), 1000), small, np.full((512, 85), -1000)], 1)
    alone = up.copy()
    alone[::4, 1, :85] = alone[::4, 1, 170:255] = 0
    dev = [torch.from_numpy(x.reshape(-1)).cuda() for x in (feat, cell, up, alone)]
    band = P.Band(torch.full((dev[0].numel(),), 0.5, device="cuda"), dev[0], dev[1], dev[0].numel())
    print("[case] cancelling terms", band.n_band, flush=True)
    got, want = (P.csc_sdf_backward(f, band, g)[torch.from_numpy(used.reshape(-1)).cuda()] for g in dev[2:])
    assert bool((want.abs().amax(1) > 0.1).all())
    wrong = int((got != want).any(1).sum())
    print("vertices off", wrong, "of", got.shape[0], flush=True)
    assert wrong == 0
