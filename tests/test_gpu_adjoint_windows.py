"""The staged adjoint at the edges of its windows, tables and projection pairs.

Tolerance: an output sums at most 131 projections x 8 samples x 8 segments of
random sign in float32; a relative rounding of 2^-24 per operation grows like the
square root of their number, 6e-8 * sqrt(8400) = 5.5e-6 relative L2.
"""
import numpy as np
import pytest
import torch

import oracle
import tt_inputs as synth
from geoms import tilted_angles
from helpers import gpu_projector, rel_l2

pytestmark = pytest.mark.gpu
TOL = 5.5e-6

# (volume, detector, rotations): 3 tilts each.  129 and 131 projections pass the
# 64-pair table of window origins (131: last pair half empty, as are those of 1 and 3);
# detectors smaller than a window, of one row, and larger than the volume's shadow;
# bricks cut on every axis (nx even: voxel pairs; odd: none)
SHAPES = {
    "pairs_past_one_table": ((8, 9, 10), (11, 12), 43),
    "unpaired_past_one_table": ((9, 8, 9), (12, 11), 43),
    "detector_below_window": ((10, 6, 9), (5, 4), 3),
    "one_detector_row": ((7, 9, 8), (1, 30), 3),
    "two_planes": ((2, 17, 3), (6, 21), 5),
    "wide_detector": ((6, 5, 4), (40, 37), 1),
}


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("n_seg", [8, 16])
@pytest.mark.parametrize("offsets", [False, True])
@pytest.mark.parametrize("name", list(SHAPES))
def test_adjoint_matches_the_oracle(name, offsets, n_seg, model):
    n, (nj, nk), n_rot = SHAPES[name]
    inner, outer = tilted_angles(n_rot, (0.0, 27.0, 45.0), span_deg=360.0)
    kw = {}
    if offsets:  # the last one moves the whole shadow off the detector
        kw = dict(joff=np.linspace(-2.0, 3.0, len(inner)), koff=np.linspace(1.5, -2.5, len(inner)))
        kw["joff"][-1] = 300.0
    og = oracle.Geometry(n, 4, inner, outer, nj, nk, n_seg, synth.lab_frame(), model=model, **kw)
    y = np.random.default_rng(5).standard_normal(og.data_shape).astype(np.float32)
    got = gpu_projector(og, device="cuda:0").adjoint(torch.from_numpy(y).cuda()).cpu().numpy()
    assert np.isfinite(got).all()
    assert rel_l2(got, oracle.adjoint(og, y.astype(np.float64))) <= TOL


@pytest.mark.parametrize("n_seg", [8, 16])
def test_a_workspace_without_room_for_splits_still_works(n_seg):
    # 129 projections of a small volume are split over blocks, each with a coefficient
    # volume of scratch at the end of the workspace; one volume less beside the smallest
    # forward batch, and the adjoint runs unsplit: the same sum in another order
    import ctypes as C

    from paper_2504_16446_amd._lib import call
    inner, outer = tilted_angles(43, (0.0, 27.0, 45.0), span_deg=360.0)
    og = oracle.Geometry((8, 9, 10), 4, inner, outer, 11, 12, n_seg, synth.lab_frame())
    P = gpu_projector(og, device="cuda:0", forward_batch=1)
    y = torch.from_numpy(np.random.default_rng(5).standard_normal(og.data_shape).astype(np.float32)).cuda()
    split = P.adjoint(y)
    volume = split.numel() * 4
    assert call("tt_workspace_bytes", P._h, 1) == P.work_bytes
    call("tt_set_workspace", P._h, C.c_void_p(P._ws.data_ptr()), P.work_bytes - volume)
    whole = P.adjoint(y)
    assert rel_l2(whole.cpu().numpy(), split.cpu().numpy()) <= TOL
    assert not torch.equal(whole, split)
