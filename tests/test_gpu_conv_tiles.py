"""Convolutions on both tile sizes (4 x 8 x 8 voxels from 256 blocks on, 4 x 4 x 8 below),
at and past the tiles' edges, against 27 float64 products on the device.

Operands are bf16, so products are exact in float32; 27 x 64 of them are summed, with at
most 2^-23 of the sum cut off per step of 32: 54 x 1.2e-7 = 6.5e-6.  The bf16 outputs add
their rounding, 2^-9 relative.
"""
import numpy as np
import pytest
import torch

from paper_2504_16446_amd import net

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (1, 4, 8, 8), (1, 5, 9, 9), (1, 32, 64, 64), (2, 33, 41, 57)])
@pytest.mark.parametrize("ci,co", [(32, 32), (32, 64), (64, 32), (64, 64)])
def test_forward_and_input_gradient(shape, ci, co):
    n, X, Y, Z = shape
    g = torch.Generator(device=DEV).manual_seed(ci + co)
    l = net.Conv3d(ci, co, DEV, np.random.default_rng(1))
    l.b.copy_(torch.randn(co, device=DEV, generator=g))
    x = torch.randn(shape + (ci,), device=DEV, generator=g).bfloat16()
    gy = torch.randn(shape + (co,), device=DEV, generator=g).bfloat16()
    w = l.w.bfloat16().double()
    pad = lambda t: torch.nn.functional.pad(t.double(), (0, 0, 1, 1, 1, 1, 1, 1))  # noqa: E731
    xp, gp = pad(x), pad(gy)
    y, gx = l.b.double(), 0.0
    for d in range(27):
        a, b, c = d // 9, d // 3 % 3, d % 3
        y = y + xp[:, a:a + X, b:b + Y, c:c + Z] @ w[d]
        gx = gx + gp[:, 2 - a:2 - a + X, 2 - b:2 - b + Y, 2 - c:2 - c + Z] @ w[d].T
    rel = lambda got, ref: float((got.double() - ref).norm() / ref.norm())  # noqa: E731
    assert rel(l.forward(x.view(torch.int16), net.BIAS_F32), y) <= 6.5e-6
    assert rel(l.forward(x.view(torch.int16), net.RELU_BF16).view(torch.bfloat16), y.clamp(min=0)) <= 2.0 ** -9
    assert rel(l.backward_input(gy.view(torch.int16), x.view(torch.int16)).view(torch.bfloat16), gx * (x > 0)) <= 2.0 ** -9
