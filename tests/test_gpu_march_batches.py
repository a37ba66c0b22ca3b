"""The march in every mix of launches that a forward batch can have, from a workspace and
into an output that hold NaN before: a ray that no launch writes, or a mapped volume
that none fills, is a NaN.

Tolerance: an output sums up to 30 samples x 8 corners (and their maps of 15 terms) in
float32; a relative rounding of 2^-24 per operation grows like the square root of their
number, 6e-8 * sqrt(240 * 15) = 3.6e-6 relative L2.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import tt_inputs as synth
from geoms import tilted_angles
from helpers import gpu_projector, rel_l2

pytestmark = pytest.mark.gpu
TOL = 3.6e-6

# (volume, detector, tilts, rotations, segments, batch), as in test_march_plan: whole LDS
# with eight segments; one launch of rings; two; rings beside slabs; rings beside
# projections gathered from memory; small batches, each with its own launches
CASES = {
    "whole_lds": ((32, 20, 17), (32, 32), (0.0, 20.0, 30.0), 20, 16, 999),
    "one_launch": ((16, 14, 15), (112, 112), (0.0, 15.0), 40, 16, 999),
    "two_launches": ((16, 14, 15), (112, 112), (0.0, 15.0), 60, 16, 999),
    "two_launches_four": ((16, 14, 15), (112, 112), (0.0, 39.0), 120, 8, 999),
    "rings_and_slabs": ((12, 11, 13), (112, 112), (0.0, 15.0, 45.0), 60, 16, 999),
    "rings_and_gathered": ((12, 11, 13), (112, 112), (0.0, 15.0, 80.0), 60, 16, 999),
    "rings_and_gathered_four": ((12, 11, 13), (112, 112), (0.0, 15.0, 80.0), 60, 8, 999),
    "small_batches": ((24, 10, 11), (40, 40), (0.0, 15.0, 45.0), 12, 16, 4),
}


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("name", list(CASES))
def test_forward(name, model):
    from paper_2504_16446_amd._lib import call
    n, (nj, nk), tilts, n_rot, n_seg, batch = CASES[name]
    inner, outer = tilted_angles(n_rot, tilts, span_deg=360.0)
    og = oracle.Geometry(n, 4, inner, outer, nj, nk, n_seg, synth.lab_frame(), model=model)
    c = np.random.default_rng(8).standard_normal(og.vol_shape).astype(np.float32)
    P = gpu_projector(og, device="cuda:0", forward_batch=batch)
    P._ws.view(torch.float32)[: P.work_bytes // 4].fill_(float("nan"))
    call("tt_set_workspace", P._h, C.c_void_p(P._ws.data_ptr()), P.work_bytes)  # (zeroes the volumes' border)
    out = torch.full(P.data_shape, float("nan"), device="cuda:0")
    got = P.forward(torch.from_numpy(c).cuda(), out=out).cpu().numpy()
    assert not np.isnan(got).any()
    assert rel_l2(got, oracle.project(og, c.astype(np.float64))) <= TOL


@pytest.mark.parametrize("n_seg", [8, 16])
@pytest.mark.parametrize("tilts, det", [((0.0, 15.0, 45.0), 112), ((0.0, 15.0, 45.0), 40), ((0.0, 20.0, 30.0), 16)])
def test_the_forward_batch_changes_no_result(tilts, det, n_seg):
    inner, outer = tilted_angles(30, tilts, span_deg=360.0)
    og = oracle.Geometry((24, 22, 20), 4, inner, outer, det, det, n_seg, synth.lab_frame())
    c = torch.from_numpy(np.random.default_rng(9).standard_normal(og.vol_shape).astype(np.float32)).cuda()
    want = gpu_projector(og, device="cuda:0").forward(c)
    for batch in (4, 16, 32):
        P = gpu_projector(og, device="cuda:0", forward_batch=batch)
        assert P.batch == batch
        assert torch.equal(P.forward(c), want), batch
