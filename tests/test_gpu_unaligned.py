"""Tensors that start at any multiple of their elements' size: tiles of other than the largest multiples of 32 tokens take
them (plain loads in place of the 16-byte DMA), in the forward pass and in both gradient kernels."""
import pytest
import torch

import paper_2502_04507_amd as sta
import synth_inputs as syn
from oracle import sta_oracle as orc
from tests import gpu_util as gu
from tests.test_gpu_backward import assert_grad_parity, oracle_backward

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def at_offset(x, elements):
    """x on the device, `elements` elements behind an aligned address."""
    y = torch.empty(x.numel() + elements, dtype=x.dtype, device=DEV)[elements:].view(x.shape)
    return y.copy_(x.to(DEV))


@pytest.mark.parametrize("elements", [1, 4])
@pytest.mark.parametrize("D,grid,tile", [(64, (1, 12, 40), (1, 4, 8)), (64, (4, 18, 24), (2, 6, 8)), (128, (1, 24, 40), (1, 8, 8)),
                                         (128, (4, 18, 24), (2, 6, 8))])
def test_tensors_at_odd_addresses(D, grid, tile, elements):
    w = syn.custom("unaligned", 1, 2, D, grid, tile, [(2, 3, 3), (1, 1, 2)], "bf16", seed=77)
    raster = (*syn.make_qkv(w), syn.make_dout(w))
    order = torch.from_numpy(orc.tile_order(w.grid, w.tile))
    q, k, v, g = (at_offset(x[:, :, order], elements) for x in raster)
    o, dq, dk, dv = (at_offset(torch.full(q.shape, float("nan"), dtype=torch.bfloat16), elements) for _ in range(4))
    assert all(x.is_contiguous() and x.data_ptr() % 16 for x in (q, k, v, g, o, dq, dk, dv))
    lse = torch.empty((1, w.H, w.N), dtype=torch.float32, device=DEV)
    sta.sta_forward_lse(q, k, v, o, lse, w.grid, w.tile, w.window_tiles)
    ws = torch.empty(sta.sta_backward_workspace_bytes(1, w.H, w.grid), dtype=torch.uint8, device=DEV)
    sta.sta_backward(q, k, v, o, g, lse, dq, dk, dv, w.grid, w.tile, w.window_tiles, ws)
    torch.cuda.synchronize()
    order = order.numpy()
    for h in range(w.H):
        gu.assert_parity(o[0, h].float().cpu().numpy(), gu.oracle_rows(w, *raster[:3], 0, h, None)[order], "h%d" % h)
        for label, got, ref in zip(("dQ", "dK", "dV"), (dq, dk, dv), oracle_backward(w, *raster, 0, h)):
            assert_grad_parity(got[0, h].float().cpu().numpy(), ref[order], "%s h%d" % (label, h))
