"""Which forward batch and whether adjoint splits a workspace gets (host, stand-in runtime)."""
import pytest

import oracle
import tt_inputs as synth
from fake_hip import scenario
from geoms import tilted_angles


def attach(F, n, ell, n_rot, n_seg, requests):
    """(batch, splits used) for each request: ("asked", b) the size that tt_workspace_bytes
    gives for batch b, ("room", b) room for b mapped volumes and nothing else."""
    inner, outer = tilted_angles(n_rot, (0.0, 15.0, 30.0, 45.0), span_deg=360.0)
    og = oracle.Geometry((n, n, n), ell, inner, outer, n, n, n_seg, synth.lab_frame())
    h = F.create(og)
    ask = lambda b: F.ok("tt_workspace_bytes", h, b)  # noqa: E731
    sizes = F.sizes(h)
    per_proj, S = sizes[7], og.n_proj
    y, g = F.buffer(4 * sizes[1]), F.buffer(4 * sizes[0])
    work = F.buffer(ask(S))
    small = 16 // (4 if n_seg == 8 else 8)
    lo, hi = 0, ask(1)  # the smallest workspace: one map tile, no splits
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if F.lib.tt_set_workspace(h, work, mid) < 0:
            lo = mid
        else:
            hi = mid
    base = hi - (per_proj * small + 255) // 256 * 256
    out = []
    for kind, b in requests:
        bytes_ = ask(b) if kind == "asked" else base + (per_proj * b + 255) // 256 * 256
        F.ok("tt_set_workspace", h, work, bytes_)
        rc, seen = F.launches("tt_adjoint", h, y, g, 0.0, None)
        assert rc == 0
        out.append((F.sizes(h)[4], any("k_add_splits" in name for name, *_ in seen)))
    return out


def _run(*args):
    return [tuple(r) for r in scenario("test_workspace_plan", "attach", *args)]


def test_a_size_that_was_asked_for_has_its_batch_and_the_splits():
    assert _run(32, 4, 15, 8, [("asked", 60), ("asked", 24), ("asked", 1)]) == [(60, True), (24, True), (4, True)]
    assert _run(48, 6, 30, 8, [("asked", 120), ("asked", 16)]) == [(120, True), (16, True)]


def test_splits_take_batches_only_where_they_save_more():
    # 32^3 / 240 projections, 56 volumes for six splits that save about 185 us: two batches
    # instead of one, or four instead of two; but not nine instead of four
    got = _run(32, 8, 60, 8, [("room", 240), ("room", 192), ("room", 72)])
    assert got == [(128, True), (128, True), (64, False)]
    # 48^3 / 120 projections, 19 volumes: three splits save about 10 us, less than a further
    # batch costs; 119 volumes leave room for them beside two batches of 64
    assert _run(48, 6, 30, 8, [("room", 119), ("room", 120), ("room", 64), ("room", 24)]) == [
        (64, True), (120, False), (64, False), (24, False)]


@pytest.mark.parametrize("n_seg", [8, 16])
def test_the_smallest_workspace_is_what_it_was_without_splits(n_seg):
    assert _run(16, 4, 16, n_seg, [("room", 16 // (4 if n_seg == 8 else 8))]) == [(16 // (4 if n_seg == 8 else 8), False)]
