"""Residuals at the ends of float32's range through the adjoint's three-piece contraction:
what the pieces cannot hold must come out as in float32.

Tolerance of the scaled residuals: as for ordinary ones, 2^-24 per operation growing like
the square root of up to 12 projections x 9 rays x 4 samples x 8 segments; scaling by a
power of two changes no rounding above 2^-126.
"""
import numpy as np
import pytest
import torch

import oracle
import tt_inputs as synth
from geoms import tilted_angles
from helpers import gpu_projector, rel_l2

pytestmark = pytest.mark.gpu
TOL = 2.0**-24 * np.sqrt(12 * 9 * 4 * 8)


def _geometry(nx, ell, n_seg, model, n_rot=4):
    inner, outer = tilted_angles(n_rot, (0.0, 27.0, 45.0), span_deg=360.0)
    return oracle.Geometry((nx, 9, 8), ell, inner, outer, 12, 13, n_seg, synth.lab_frame(), model=model)


@pytest.mark.parametrize("exponent", [-118, -100, 100, 122])
@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("nx", [8, 9])
@pytest.mark.parametrize("ell, n_seg", [(4, 8), (8, 8), (8, 16), (8, 12)])
def test_scaled_residuals(ell, n_seg, nx, model, exponent):
    og = _geometry(nx, ell, n_seg, model)
    y = np.random.default_rng(11).standard_normal(og.data_shape).astype(np.float32)
    scaled = torch.from_numpy(np.ldexp(y, exponent)).cuda()
    got = gpu_projector(og, device="cuda:0").adjoint(scaled).cpu().numpy().astype(np.float64)
    assert rel_l2(np.ldexp(got, -exponent), oracle.adjoint(og, y.astype(np.float64))) <= TOL


@pytest.mark.parametrize("n_seg", [8, 16])
def test_finite_residuals_above_the_largest_bf16(n_seg):
    # one projection along an axis, one segment: each voxel's Q is one detector value, and
    # no partial sum leaves float32 (the constants are below 1)
    og = oracle.Geometry((8, 8, 8), 4, np.zeros(1), np.zeros(1), 8, 8, n_seg, synth.lab_frame())
    y = np.zeros(og.data_shape, np.float32)
    y[..., 1] = 3.396e38
    assert np.abs(og.B()).max() < 1.0
    got = gpu_projector(og, device="cuda:0").adjoint(torch.from_numpy(y).cuda()).cpu().numpy().astype(np.float64)
    assert rel_l2(got / 2.0**100, oracle.adjoint(og, y.astype(np.float64) / 2.0**100)) <= TOL


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("nx", [8, 9])
@pytest.mark.parametrize("ell, n_seg, n_rot", [(4, 8, 4), (8, 8, 4), (8, 16, 4), (8, 8, 43)])  # (129 projections: splits)
def test_an_infinite_residual_is_infinite_where_it_reaches(ell, n_seg, n_rot, nx, model, precision):
    og = _geometry(nx, ell, n_seg, model, n_rot)
    y = np.random.default_rng(12).standard_normal(og.data_shape).astype(np.float32)
    at = (2, 6, 6, 1)
    y[at] = np.inf
    unit = np.zeros(og.data_shape)
    unit[at] = 1.0
    reach = oracle.adjoint(og, unit)
    P = gpu_projector(og, device="cuda:0", map_precision=precision)
    got = P.adjoint(torch.from_numpy(y).cuda()).cpu().numpy()
    clear = np.abs(reach) > 1e-4 * np.abs(reach).max()  # beside them, weights and constants of rounding size
    assert clear.sum() > 20
    assert np.array_equal(got[clear], np.copysign(np.inf, reach[clear]).astype(np.float32))
    # voxels that neither this ray nor its neighbours reach (a weight of rounding size is
    # enough for an infinity)
    unit[at[0], 5:8, 5:8, at[3]] = 1.0
    away = (oracle.adjoint(og, unit) == 0.0).all(axis=-1)
    assert away.sum() > 100 and np.isfinite(got[away]).all()
    y[at] = 0.0
    want = oracle.adjoint(og, y.astype(np.float64))
    assert rel_l2(got[away], want[away]) <= (TOL if precision == "fp32" else 2.0**-8)


def test_an_undefined_residual_is_undefined_where_it_reaches():
    og = _geometry(8, 8, 8, "trilinear")
    y = np.random.default_rng(13).standard_normal(og.data_shape).astype(np.float32)
    at = (2, 6, 6, 1)
    unit = np.zeros(og.data_shape)
    unit[at] = 1.0
    reach = np.abs(oracle.adjoint(og, unit)).max(axis=-1)
    unit[at[0], 5:8, 5:8, at[3]] = 1.0
    away = (oracle.adjoint(og, unit) == 0.0).all(axis=-1)
    y[at] = np.nan
    got = gpu_projector(og, device="cuda:0").adjoint(torch.from_numpy(y).cuda()).cpu().numpy()
    assert np.isnan(got[reach > 1e-4 * reach.max()]).all() and np.isfinite(got[away]).all()
