"""Every value of an adjoint is written by its own call: the output and all scratch hold NaN
before it (of one bit pattern the output, of another the scratch, so that a failure says
which kernel missed a value).

Tolerance: an output sums at most 131 projections x 8 samples x 8 segments of random sign
in float32; a relative rounding of 2^-24 per operation grows like the square root of
their number, 6e-8 * sqrt(8400) = 5.5e-6 relative L2.  bf16 tier: two factors rounded to
2^-9 each.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from adjoint_shapes import SHAPES, geometry
from helpers import gpu_projector, rel_l2

pytestmark = pytest.mark.gpu
TOL = {"fp32": 5.5e-6, "bf16": 2.0**-8}
OUT, SCRATCH = 0x7FC00AAA, 0x7FC00BBB


def _adjoint(og, y, precision):
    from paper_2504_16446_amd._lib import call
    P = gpu_projector(og, device="cuda:0", map_precision=precision, forward_batch=1)
    P._ws.view(torch.int32).fill_(SCRATCH)
    call("tt_set_workspace", P._h, C.c_void_p(P._ws.data_ptr()), P.work_bytes)
    out = torch.empty(P.vol_shape, device="cuda:0")
    out.view(torch.int32).fill_(OUT)
    return P.adjoint(y, out=out).cpu().numpy()


def _check(name, ell, n_seg, model, precision="fp32"):
    og = geometry(name, ell, n_seg, model)
    y = np.random.default_rng(5).standard_normal(og.data_shape).astype(np.float32)
    got = _adjoint(og, torch.from_numpy(y).cuda(), precision)
    bits = got.view(np.int32)
    assert not np.isnan(got).any(), f"{(bits == OUT).sum()} values not written, {np.isnan(got).sum()} NaN"
    assert rel_l2(got, oracle.adjoint(og, y.astype(np.float64))) <= TOL[precision]


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("ell, n_seg", [(4, 8), (4, 16), (8, 8), (8, 16)])
@pytest.mark.parametrize("name", list(SHAPES))
def test_adjoint(name, ell, n_seg, model):
    _check(name, ell, n_seg, model)


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("ell, n_seg", [(10, 8), (12, 8), (12, 16), (6, 8)])
@pytest.mark.parametrize("name", ["paired_129", "offsets_131"])
def test_adjoint_of_other_orders(name, ell, n_seg, model):
    _check(name, ell, n_seg, model)


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
@pytest.mark.parametrize("ell, n_seg", [(4, 8), (8, 8), (8, 16), (12, 8)])
@pytest.mark.parametrize("name", ["paired_129", "paired_131", "unpaired_129", "offsets_131"])
def test_bf16_tier(name, ell, n_seg, model):
    _check(name, ell, n_seg, model, "bf16")


@pytest.mark.parametrize("model", ["trilinear", "joseph"])
def test_projectors_in_turn_on_the_same_memory(model):
    # the second projector's buffers are the first one's: what it does not write would be
    # the first one's numbers
    other = "joseph" if model == "trilinear" else "trilinear"
    a, b = geometry("paired_129", 4, 8, other), geometry("paired_129", 4, 8, model)
    y = np.random.default_rng(6).standard_normal(a.data_shape).astype(np.float32)
    for og in (a, b, a, b):
        got = gpu_projector(og, device="cuda:0").adjoint(torch.from_numpy(y).cuda()).cpu().numpy()
        assert rel_l2(got, oracle.adjoint(og, y.astype(np.float64))) <= TOL["fp32"]
