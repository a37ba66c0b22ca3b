"""The adjoint at sample spacings from 2 to 0.1 voxels: up to three samples of a ray
within a voxel's cube, a remainder beyond them, and the unrolled loop with each remainder.

Tolerance: an output sums up to 12 projections x 9 rays x 2 sqrt(3) / step samples in
float32; a relative rounding of 2^-24 per operation grows like the square root of their
number.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import tt_inputs as synth
from geoms import tilted_angles
from helpers import gpu_projector, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("step", [2.0, 0.55, 0.5, 0.4, 0.34, 0.3, 0.27, 0.1])
@pytest.mark.parametrize("nx", [10, 11])  # pairs of voxels, and none
@pytest.mark.parametrize("ell, n_seg", [(4, 8), (8, 8), (8, 16), (10, 8)])
def test_adjoint(ell, n_seg, nx, step):
    inner, outer = tilted_angles(4, (0.0, 27.0, 45.0), span_deg=360.0)
    og = oracle.Geometry((nx, 9, 8), ell, inner, outer, 12, 13, n_seg, synth.lab_frame(), step=step)
    y = np.random.default_rng(3).standard_normal(og.data_shape).astype(np.float32)
    got = gpu_projector(og, device="cuda:0").adjoint(torch.from_numpy(y).cuda()).cpu().numpy()
    tol = 2.0**-24 * math.sqrt(12 * 9 * max(1.0, 2 * math.sqrt(3) / step))
    assert rel_l2(got, oracle.adjoint(og, y.astype(np.float64))) <= tol
