"""Weight and bias gradients at the edges of the 2 x 8 x 8-voxel tiles and of the chunks.

Inputs are bf16-representable, so products are exact in float32.  The MFMA cuts its
float32 accumulator off: at most 2^-23 of the partial sum per step of 32 voxels, against
sums of random sign that grow like the square root of the voxels, gives (voxels / 32)
steps x 2^-23 / 2 on average: 1.2e-5 for the largest case here (6336 voxels in one chunk
at worst), 2e-6 and less for the others.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import conv as oconv
from paper_2504_16446_amd import net

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _bits(a):
    u = np.ascontiguousarray(a, dtype=np.float32).view(np.uint32) >> 16
    return torch.from_numpy(u.astype(np.uint16).view(np.int16)).to(DEV)


# one voxel; below, at and past a tile in every axis; several tiles per chunk (1 x 2 x 8 x 8
# tiles need 337 and more); a batch
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (1, 2, 8, 8), (1, 3, 9, 7), (2, 1, 8, 17), (3, 4, 16, 33)])
@pytest.mark.parametrize("ci,co", [(32, 32), (32, 64), (64, 32), (64, 64)])
def test_weight_gradient(shape, ci, co):
    rng = np.random.default_rng(ci + co)
    x = oracle.bf16(rng.standard_normal(shape + (ci,)))
    gy = oracle.bf16(rng.standard_normal(shape + (co,)))
    l = net.Conv3d(ci, co, DEV, rng)
    need = net.lib().tt_conv3d_wgrad_work_bytes(ci, co, *shape)
    work = torch.full(((need + 3) // 4,), float("nan"), device=DEV)
    l.backward_weights(_bits(x), _bits(gy), work)
    gw, gb = oconv.conv3d_wgrad(x, gy), gy.reshape(-1, co).sum(0)
    assert np.linalg.norm(l.gw.cpu().numpy().reshape(gw.shape) - gw) <= 1.2e-5 * np.linalg.norm(gw)
    assert np.linalg.norm(l.gb.cpu().numpy() - gb) <= 1.2e-5 * np.linalg.norm(gb)


def test_weight_gradient_with_several_tiles_per_chunk():
    # 6 x 24 x 32 x 32 voxels: 1152 tiles over 168 chunks; against the gradient as 27 float64 products
    g = torch.Generator(device=DEV).manual_seed(3)
    x = torch.randn((6, 24, 32, 32, 32), device=DEV, generator=g).bfloat16()
    gy = torch.randn((6, 24, 32, 32, 64), device=DEV, generator=g).bfloat16()
    l = net.Conv3d(32, 64, DEV, np.random.default_rng(0))
    need = net.lib().tt_conv3d_wgrad_work_bytes(32, 64, *x.shape[:4])
    l.backward_weights(x.view(torch.int16), gy.view(torch.int16), torch.empty((need + 3) // 4, device=DEV))
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1, 1, 1))
    gd = gy.double().reshape(-1, 64)
    for d in range(27):
        a, b, c = d // 9, d // 3 % 3, d % 3
        ref = xp[:, a:a + 24, b:b + 32, c:c + 32].reshape(-1, 32).T @ gd
        assert float((l.gw[d].double() - ref).norm() / ref.norm()) <= 1.2e-5
    assert float((l.gb.double() - gd.sum(0)).norm() / gd.sum(0).norm()) <= 1.2e-5
