"""The permutation kernels on both sides of the size from which they read with streaming loads (256 MB of source)."""
import pytest
import torch

import paper_2502_04507_amd as sta
from oracle import sta_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GRID, TILE, D = (6, 16, 24), (6, 8, 8), 64
SLICE = 2304 * D                                             # elements of one head


@pytest.mark.parametrize("above", [False, True], ids=["at", "above"])
@pytest.mark.parametrize("src,dst", [(torch.bfloat16, torch.bfloat16), (torch.float32, torch.bfloat16),
                                     (torch.bfloat16, torch.float32), (torch.float32, torch.float32)])
def test_permutation_at_the_streaming_size(src, dst, above):
    heads = (256 << 20) // (SLICE * src.itemsize) + (1 if above else 0)
    g = torch.Generator(device=DEV).manual_seed(3)
    x = torch.randn((1, heads, 2304, D), generator=g, device=DEV, dtype=torch.float32).to(src)
    order = torch.from_numpy(orc.tile_order(GRID, TILE)).to(DEV)
    y = torch.full(x.shape, float("nan"), dtype=dst, device=DEV)
    sta.sta_tile_permute(x, y, GRID, TILE)
    assert torch.equal(y, x[:, :, order].to(dst))
    z = torch.full(x.shape, float("nan"), dtype=dst, device=DEV)
    sta.sta_untile(x, z, GRID, TILE)
    assert torch.equal(z[:, :, order], x.to(dst))
