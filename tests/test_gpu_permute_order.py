"""The permutation kernels where their split over workgroups can go wrong: full rounds of eight rows of tiles and what is left over, tiles
that end inside a workgroup's share, one and two pieces per lane, and more workgroups than one dimension of a grid holds."""
import numpy as np
import pytest
import torch

import paper_2502_04507_amd as sta
from oracle import sta_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TYPES = [(torch.bfloat16, torch.bfloat16), (torch.float32, torch.bfloat16), (torch.bfloat16, torch.float32),
         (torch.float32, torch.float32)]


@pytest.mark.parametrize("src,dst", TYPES, ids=["b-b", "f-b", "b-f", "f-f"])
@pytest.mark.parametrize("slices,D,grid,tile", [
    (1, 64, (1, 32, 24), (1, 4, 8)),        # eight rows: one full round, a piece per lane fills the workgroup
    (3, 64, (1, 24, 24), (1, 4, 8)),        # 18 rows: two rounds and two rows
    (1, 64, (1, 12, 24), (1, 4, 8)),        # three rows: no round
    (5, 72, (3, 10, 14), (3, 5, 7)),        # 945 pieces a tile: the last workgroup of a tile is partly empty
    (7, 64, (2, 9, 12), (2, 3, 12)),    # one tile per row, 576 pieces
    (2, 8, (4, 16, 33), (1, 1, 1)),         # one piece a tile
    (9, 128, (6, 16, 8), (6, 8, 8)),        # 6144 pieces a tile
], ids=str)
def test_split_over_workgroups(slices, D, grid, tile, src, dst):
    N = int(np.prod(grid))
    g = torch.Generator().manual_seed(11)
    x = torch.randn((1, slices, N, D), generator=g).to(src).to(DEV)
    order = torch.from_numpy(orc.tile_order(grid, tile)).to(DEV)
    y = torch.full(x.shape, float("nan"), dtype=dst, device=DEV)
    sta.sta_tile_permute(x, y, grid, tile)
    assert torch.equal(y, x[:, :, order].to(dst))
    z = torch.full(x.shape, float("nan"), dtype=dst, device=DEV)
    sta.sta_untile(x, z, grid, tile)
    assert torch.equal(z[:, :, order], x.to(dst))


def test_more_workgroups_than_a_grid_is_wide():
    grid, tile, D = (8, 1024, 2050), (1, 2, 1), 8            # 8.4 million tiles; 2^23 workgroups along x
    x = torch.arange(8 * 1024 * 2050 * D, device=DEV, dtype=torch.int32).to(torch.int16).view(1, 1, -1, D).view(torch.bfloat16)
    want = x.view(torch.int16).view(8, 512, 2, 2050, D).permute(0, 1, 3, 2, 4).reshape(x.shape)
    y = torch.zeros_like(x)
    sta.sta_tile_permute(x, y, grid, tile)
    assert torch.equal(y.view(torch.int16), want)
    z = torch.zeros_like(x)
    sta.sta_untile(y, z, grid, tile)
    assert torch.equal(z.view(torch.int16), x.view(torch.int16))
