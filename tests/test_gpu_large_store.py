"""A store of more bricks than the sign pass has wavefronts (2^18), so that they go
round a second time: every copy of a mesh in a batch against the mesh alone."""
import pytest

import meshgen
from meshgen import Grid

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1903_00353_amd as P  # noqa: E402


@pytest.mark.parametrize("kept", [False, True])
def test_copies_past_the_sign_pass_grid(kept):
    v, f = meshgen.icosphere(4)
    g = Grid.unit(256, 3)
    alone = P.Batch([(v, f)], [g], backward=False)
    alone.step()
    alone.check()
    want = alone.band(0)
    copies = (1 << 18) // int(alone.f.info()["n_bricks"]) + 2
    print("[case] copies", copies, "kept" if kept else "filled", flush=True)
    B = P.Batch([(v, f)] * copies, [g] * copies, backward=False, headroom=1.0)
    assert int(B.f.info()["n_bricks"]) > 1 << 18
    if kept:  # the store emptied by the first scan's sign pass serves the second
        B.step()
        B.step()
        B.check()
    else:
        nbytes, _ = P.csc_scan_convert_workspace(B.f)
        P.csc_scan_convert_batched(B.f, torch.empty(nbytes, dtype=torch.uint8, device="cuda"), B.out, B.band_off)
    off = B.band_off.cpu().tolist()
    assert off == [k * want[0].numel() for k in range(copies + 1)]
    for m in range(copies):
        assert all(torch.equal(a, b) for a, b in zip(B.band(m), want))
