"""The forward march over rings of staged planes, at the edges of its plans.

Tolerance: an output sums at most 30 samples x 8 corners x 15 channels of random sign
in float32, 6e-8 * sqrt(3600) = 3.6e-6 relative L2; a position inside a plane's box of
at most 32 voxels is rounded by 1.9e-6 of a voxel at most: 5.5e-6 together.
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

# (volume, detector, rotations, tilts).  Blocks of 16 x 16 rays: up to 256 take a
# compute unit's whole LDS, up to 8191 are one launch, more are two launches by LDS
# size with the projections of large planes on slabs; tilts of 80 degrees run along z,
# where no ring is planned
SHAPES = {
    "one_block_per_unit": ((12, 14, 10), (20, 18), 8, (0.0, 27.0, 45.0)),
    "one_launch": ((10, 9, 12), (70, 66), 7, (0.0, 20.0, 30.0)),
    "two_launches": ((9, 10, 8), (256, 256), 11, (0.0, 27.0, 45.0)),
    "one_plane_x": ((1, 20, 3), (17, 30), 5, (0.0, 30.0)),
    "one_plane_y": ((20, 1, 3), (30, 17), 5, (0.0, 30.0)),
    "one_voxel": ((1, 1, 1), (5, 16), 4, (0.0, 30.0)),
    "along_z": ((8, 9, 21), (33, 15), 4, (0.0, 80.0)),
}


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("n_seg", [8, 16])
@pytest.mark.parametrize("offsets", [False, True])
@pytest.mark.parametrize("name", list(SHAPES))
def test_forward_matches_the_oracle(name, offsets, n_seg, model):
    n, (nj, nk), n_rot, tilts = SHAPES[name]
    inner, outer = tilted_angles(n_rot, tilts, span_deg=360.0)
    kw = {}
    if offsets:  # the last one moves the whole shadow off the detector
        kw = dict(joff=np.linspace(-2.0, 3.0, len(inner)), koff=np.linspace(1.5, -2.5, len(inner)))
        kw["joff"][-1] = 600.0
    og = oracle.Geometry(n, 4, inner, outer, nj, nk, n_seg, synth.lab_frame(), model=model, **kw)
    c = np.random.default_rng(6).standard_normal(og.vol_shape).astype(np.float32)
    want = oracle.project(og, c.astype(np.float64))
    x = torch.from_numpy(c).cuda()
    # all projections in one pass, and in the smallest passes
    for kw in ({}, {"forward_batch": 16 // min(n_seg // 2, 8)}):
        got = gpu_projector(og, device="cuda:0", **kw).forward(x).cpu().numpy()
        assert np.isfinite(got).all()
        assert rel_l2(got, want) <= TOL
