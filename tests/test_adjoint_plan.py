"""Which adjoint kernel a geometry runs, from its launches on a stand-in runtime
(template arguments: unique segments, 16-coefficient tiles, bf16 tier, Joseph, paired,
four waves per SIMD, many samples per ray)."""
import pytest

import oracle
import tt_inputs as synth
from fake_hip import scenario
from geoms import tilted_angles


def adjoint_launches(F, n, ell, n_rot, n_seg, model, offsets, step):
    inner, outer = tilted_angles(n_rot, (0.0, 15.0, 30.0, 45.0), span_deg=360.0)
    kw = dict(joff=[0.5] * len(inner), koff=[0.25] * len(inner)) if offsets else {}
    og = oracle.Geometry((n, n, n), ell, inner, outer, n, n, n_seg, synth.lab_frame(), model=model, step=step, **kw)
    h = F.create(og, model)
    F.workspace(h, 1)
    s = F.sizes(h)
    rc, seen = F.launches("tt_adjoint", h, F.buffer(4 * s[1]), F.buffer(4 * s[0]), 0.0, None)
    assert rc == 0
    return [name for name, *_ in seen]


def _kernel(names, up, mt, *flags):
    name = f"k_backproject_winILi{up}ELi{mt}E" + "".join(f"Lb{int(f)}E" if isinstance(f, bool) else f"Li{f}E" for f in flags)
    assert any(name in k for k in names), (name, names)


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("n, deep", [(48, False), (56, False), (64, True), (72, False), (80, True), (96, True)])
def test_unpaired_adjoints_of_four_segments_and_48_coefficients(n, deep, model):
    # blocks of 4 x 8 x 8 voxels per compute unit: 2, 3, 4, 6, 8, 14; four at a time where that
    # saves a round or there are many
    names = scenario("test_adjoint_plan", "adjoint_launches", n, 8, 30, 8, model, True, 1.0)
    _kernel(names, 4, 3, False, model == "joseph", False, deep)


def test_paired_adjoints_keep_three_waves():
    names = scenario("test_adjoint_plan", "adjoint_launches", 64, 8, 30, 8, "trilinear", False, 1.0)
    _kernel(names, 4, 3, False, False, True, False)


def random_frames(F, n_seg, nx, model):
    import numpy as np
    r = np.random.default_rng(n_seg + nx)
    og = oracle.Geometry((nx, 40, 40), 8, r.uniform(0, 2 * np.pi, 400), r.uniform(0, np.pi, 400), 60, 60, n_seg,
                         synth.lab_frame(), model=model)
    h = F.create(og, model)
    F.workspace(h, 1)
    s = F.sizes(h)
    rc, seen = F.launches("tt_adjoint", h, F.buffer(4 * s[1]), F.buffer(4 * s[0]), 0.0, None)
    return rc, [name for name, *_ in seen]


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("nx", [40, 41])
@pytest.mark.parametrize("n_seg", [8, 16])
def test_windows_of_any_orientation_fit(n_seg, nx, model):
    # up to eight unique segments have no other kernel
    rc, names = scenario("test_adjoint_plan", "random_frames", n_seg, nx, model)
    assert rc == 0 and any("k_backproject_win" in k for k in names)


@pytest.mark.parametrize("n_seg, up, deep", [(8, 4, True), (16, 8, False)])
@pytest.mark.parametrize("offsets", [False, True])
def test_small_steps_unroll_the_samples_of_a_ray(offsets, n_seg, up, deep):
    names = scenario("test_adjoint_plan", "adjoint_launches", 64, 8, 30, n_seg, "trilinear", offsets, 0.25)
    _kernel(names, up, 3, False, False, not offsets, deep, True)
    names = scenario("test_adjoint_plan", "adjoint_launches", 64, 8, 30, n_seg, "trilinear", offsets, 0.8)
    assert not any("Lb0ELb1EEEv" in k or "Lb1ELb1EEEv" in k for k in names), names


def edge_shape(F, name, ell, n_seg, model):
    from adjoint_shapes import geometry
    og = geometry(name, ell, n_seg, model)
    h = F.create(og, model)
    F.workspace(h, 1)
    s = F.sizes(h)
    rc, seen = F.launches("tt_adjoint", h, F.buffer(4 * s[1]), F.buffer(4 * s[0]), 0.0, None)
    assert rc == 0
    return [name for name, *_ in seen]


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("ell, n_seg, up, mt", [(4, 8, 4, 1), (8, 8, 4, 3), (8, 16, 8, 3)])
@pytest.mark.parametrize("name, paired, split", [("paired_129", True, True), ("unpaired_129", False, True),
                                                 ("offsets_131", False, True), ("one_projection", True, False)])
def test_edge_shapes_run_what_they_are_for(name, paired, split, ell, n_seg, up, mt, model):
    names = scenario("test_adjoint_plan", "edge_shape", name, ell, n_seg, model)
    _kernel(names, up, mt, False, model == "joseph", paired, False)
    assert any("k_add_splits" in k for k in names) == split
