"""Tile of a convolution by its blocks (host, stand-in runtime)."""
import pytest

from fake_hip import scenario


def conv_kernel(F, n, tile, ci, co):
    b = F.buffer(1 << 16)
    rc, seen = F.launches("tt_conv3d", 0, ci, co, b, b, b, None, b, n, tile, tile, tile, None)
    assert rc == 0 and len(seen) == 1, (rc, F.lib.tt_last_error())
    return seen[0][:2]


@pytest.mark.parametrize("n, tile, wide, blocks", [(1, 32, False, 256), (1, 41, False, 726), (1, 48, True, 432),
                                                   (2, 36, True, 450)])
@pytest.mark.parametrize("ci, co", [(32, 32), (32, 64), (64, 32), (64, 64)])
def test_wide_tile_from_400_blocks_on(ci, co, n, tile, wide, blocks):
    name, grid = scenario("test_conv_plan", "conv_kernel", n, tile, ci, co)
    assert f"k_convILi{ci}ELi{co}ELi0ELi{8 if wide else 4}E" in name and grid == blocks
