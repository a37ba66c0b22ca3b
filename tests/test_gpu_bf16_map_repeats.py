"""The bf16 map gives the same bits on every run (its MFMA chain is one instruction)."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ell", [2, 4, 8, 10])  # 16, 16, 48 and 80 padded coefficients: odd multiples of 16
def test_repeated_bf16_forwards_are_equal(ell):
    from paper_2504_16446_amd.projector import Projector
    inner = np.arange(40) * (2 * math.pi / 40)
    P = Projector((96, 96, 96), ell, inner, np.full(40, 0.3), 96, 96, 16, device="cuda:0", map_precision="bf16")
    c = torch.randn(P.vol_shape, device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(1))
    first = P.forward(c)
    for _ in range(3):
        assert torch.equal(P.forward(c), first)
