"""Launches of the march for one forward batch, on a stand-in runtime: rings of staged
planes in one launch or two, slabs, or both, by the blocks and the projections of the batch."""
import pytest

import oracle
import tt_inputs as synth
from fake_hip import scenario
from geoms import tilted_angles


def march_launches(F, n, det, tilts, n_rot, n_seg, batch):
    inner, outer = tilted_angles(n_rot, tilts, span_deg=360.0)
    og = oracle.Geometry((n, n, n), 2, inner, outer, det, det, n_seg, synth.lab_frame())
    h = F.create(og)
    F.workspace(h, batch)
    s = F.sizes(h)
    rc, seen = F.launches("tt_project", h, F.buffer(4 * s[0]), F.buffer(4 * s[1]))
    assert rc == 0
    out = []
    for name, blocks, lds in seen:
        if "k_map" in name:
            out.append([])
        else:
            out[-1].append(("ring" if "k_march_ring" in name else "slab", blocks, lds))
    return s[4], out


def _run(*args):
    return scenario("test_march_plan", "march_launches", *args)


FLAT, STEEP, GATHERED = (0.0, 15.0), (0.0, 15.0, 45.0), (0.0, 15.0, 80.0)


@pytest.mark.parametrize("n_seg", [8, 16])
def test_a_small_batch_runs_its_rings_in_one_launch(n_seg):
    # 49 blocks per projection; the batches of 16 hold 784 blocks, all of them 17640
    batch, seen = _run(24, 112, STEEP, 120, n_seg, 16)
    assert batch == 16 and len(seen) == 23
    kinds = [[kind for kind, *_ in launches] for launches in seen]
    assert all(k in (["ring"], ["slab"], ["ring", "slab"]) for k in kinds)
    assert kinds.count(["ring"]) >= 15 and (n_seg == 8 or ["slab"] in kinds or ["ring", "slab"] in kinds)
    batch, seen = _run(24, 112, STEEP, 120, n_seg, 360)
    assert batch == 360 and len(seen) == 1 and 2 <= len(seen[0]) <= 3


@pytest.mark.parametrize("n_seg", [8, 16])
def test_which_projections_run_on_rings_does_not_depend_on_the_batch(n_seg):
    # a projection on a ring or on slabs is rounded differently: 360 x 16 blocks, too few for both
    for batch in (8, 360):
        _, seen = _run(20, 60, STEEP, 120, 16, batch)
        assert {kind for launches in seen for kind, *_ in launches} == {"slab"}
    # and enough
    for batch in (8, 360):
        _, seen = _run(24, 112, STEEP, 120, 16, batch)
        assert {kind for launches in seen for kind, *_ in launches} == {"ring", "slab"}


@pytest.mark.parametrize("n_seg, n_rot, launches", [(16, 40, 1), (16, 60, 2), (8, 60, 1), (8, 120, 2)])
def test_two_launches_from_4096_or_8192_blocks_on(n_seg, n_rot, launches):
    # 49 blocks per projection: 3920, 5880 and 11760, with rings of both sizes
    _, seen = _run(16, 112, FLAT if n_seg == 16 else (0.0, 39.0), n_rot, n_seg, 999)
    assert [len(b) for b in seen] == [launches]
    assert all(kind == "ring" for kind, *_ in seen[0])
    assert len({lds for *_, lds in seen[0]}) == launches


@pytest.mark.parametrize("n_seg", [8, 16])
def test_up_to_one_block_per_unit_takes_the_whole_lds(n_seg):
    _, seen = _run(32, 32, (0.0, 20.0, 30.0), 20, n_seg, 999)  # 240 blocks
    assert len(seen[0]) == 1
    kind, blocks, lds = seen[0][0]
    assert kind == "ring" and blocks == 240 and lds > 80 * 1024


@pytest.mark.parametrize("n_seg", [8, 16])
def test_rings_and_gathered_projections_in_one_batch(n_seg):
    _, seen = _run(12, 112, GATHERED, 60, n_seg, 999)  # 8820 blocks
    kinds = [kind for kind, *_ in seen[0]]
    assert kinds.count("slab") == 1 and kinds.count("ring") >= 1


def test_sixteen_segments_stay_on_slabs():
    _, seen = _run(12, 30, FLAT, 8, 30, 999)
    assert [k for k, *_ in seen[0]] == ["slab"]
