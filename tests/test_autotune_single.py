"""The schedule of one mesh is chosen on the launches that a real call makes."""
import sys
import types

import paper_1903_00353_amd as P
from paper_1903_00353_amd import autotune


def test_single_mesh_search_scores_untimed_calls():
    """Stage by stage (kinds one after another) 32 rows and grid 1 are fastest, in the one
    launch of an untimed call 64 rows of faces, 16 of edges and grid 3."""
    def measure(opt, reps):
        t = {k: 0.0 for k in autotune.FORWARD_STAGES}
        for k, kind in enumerate(autotune.KIND_STAGES):
            t[kind] = 1.0 if opt.small_rows[k] == 32 else 2.0
            t[kind + "_big"] = 0.0
        t["sign"] = 0.1 * opt.scan_grid
        t["step"] = (5.0 - (opt.small_rows[0] == 64) - (opt.small_rows[1] == 16) - (opt.scan_grid == 3)
                     + abs(opt.absorb_cells - 0.05))
        return t

    (rows, grid, absorb, geom), timings = autotune._search(measure, P.make_options(absorb_cells=0.05), 1)
    assert rows[:2] == (64, 16) and grid == 3 and absorb == 0.05 and geom == 0
    assert abs(timings["grid=3"] - 2.0) < 1e-6


def test_tune_single_measures_the_untimed_scan(monkeypatch):
    """Each candidate is timed by stages and as an untimed call."""
    seen = []
    torch = types.SimpleNamespace(
        empty=lambda *a, **k: None, zeros=lambda *a, **k: None, uint8=0, float32=0, int32=0, int64=0)
    monkeypatch.setitem(sys.modules, "torch", torch)
    monkeypatch.setattr(autotune, "signature", lambda *a: "sig")
    feats = types.SimpleNamespace(free=lambda: None)
    monkeypatch.setattr(P, "csc_build_features", lambda *a: feats)
    monkeypatch.setattr(P, "csc_scan_convert_workspace", lambda f: (1, 1))
    monkeypatch.setattr(P, "csc_scan_convert", lambda f, *a, **k: seen.append("scan"))
    monkeypatch.setattr(autotune, "_stage_times",
                        lambda run, reps: run() or {k: 1.0 for s in autotune.FORWARD_STAGES for k in (s, s + "_big")})
    monkeypatch.setattr(autotune, "_step_time", lambda run, reps: run() or 1.0)
    monkeypatch.setattr(autotune, "save", lambda *a: None)
    mesh = types.SimpleNamespace(shape=(4, 3), device="cpu")
    choice, timings = autotune.tune_single(mesh, mesh, None, use_cache=False)
    assert len(seen) == 2 * len([k for k in timings])
    assert timings["rows=8"]["step"] == 1.0


def test_choices_of_other_kernels_are_not_taken(monkeypatch):
    """The cache's keys differ from those of choices made before the three kinds shared
    their launches (key version 6)."""
    import torch
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda i: types.SimpleNamespace(gcnArchName="gfx950", name=""))
    grid = types.SimpleNamespace(n=(64, 64, 64), band=3.0)
    version = autotune.signature([1000], [grid]).rsplit("|v", 1)[1]
    assert int(version) > 6
