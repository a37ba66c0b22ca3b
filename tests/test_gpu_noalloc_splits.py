"""tt_loss_grad_noalloc against tt_loss_grad where the adjoint of a small volume is split
over the projections: equal bit for bit where both have room for the splits' sums, equal
up to the order of summation where only one has.

Tolerance of the latter: sums over 129 projections x 9 rays x 4 samples x 8 segments of a
residual of order one, 2^-24 per operation growing like the square root of their number,
on both sides.
"""
import ctypes as C

import pytest
import torch

import oracle
import tt_inputs as synth
from geoms import tilted_angles
from helpers import gpu_projector, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _noalloc(P, c, data):
    from paper_2504_16446_amd._lib import call
    loss = torch.full((1,), float("nan"), dtype=torch.float64, device=DEV)
    grad = torch.full(P.vol_shape, float("nan"), dtype=torch.float32, device=DEV)
    P._bind_stream()
    call("tt_loss_grad_noalloc", P._h, C.c_void_p(c.data_ptr()), C.c_void_p(data.data_ptr()), None, 1e-3,
         C.c_void_p(loss.data_ptr()), C.c_void_p(grad.data_ptr()), None)
    return loss, grad


@pytest.mark.parametrize("n_seg", [8, 16])
@pytest.mark.parametrize("model", ["trilinear", "joseph"])
def test_same_and_other_split(n_seg, model):
    from paper_2504_16446_amd._lib import call
    inner, outer = tilted_angles(43, (0.0, 27.0, 45.0), span_deg=360.0)
    og = oracle.Geometry((8, 9, 10), 4, inner, outer, 11, 12, n_seg, synth.lab_frame(), model=model)
    P = gpu_projector(og, device=DEV, forward_batch=1)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(21)
    c = torch.randn(P.vol_shape, device=DEV, generator=gen)
    data = torch.randn(P.data_shape, device=DEV, generator=gen)
    loss, grad = _noalloc(P, c, data)
    ref_loss, ref_grad, _ = P.loss_grad(c, data, None, 1e-3)
    assert torch.equal(grad, ref_grad) and loss.item() == ref_loss.item()
    # the smallest workspace and one volume less than the splits need
    call("tt_set_workspace", P._h, C.c_void_p(P._ws.data_ptr()), P.work_bytes - 4 * grad.numel())
    whole_loss, whole, _ = P.loss_grad(c, data, None, 1e-3)
    assert not torch.equal(grad, whole)
    assert rel_l2(grad.cpu(), whole.cpu()) <= 2 * 2.0**-24 * (129 * 9 * 4 * 8) ** 0.5
    assert abs(loss.item() / whole_loss.item() - 1) <= 1e-12
