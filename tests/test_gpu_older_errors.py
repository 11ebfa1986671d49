"""An error that an earlier call of the program left for hipGetLastError is that call's: no entry point takes it for one of its own."""
import ctypes

import pytest
import torch

import paper_2502_04507_amd as sta

pytestmark = pytest.mark.gpu
GRID, TILE, WINDOWS = (1, 12, 16), (1, 4, 8), [(1, 3, 1)]


def bf16(offset=0):
    x = torch.zeros(GRID[1] * GRID[2] * 64 + offset, dtype=torch.bfloat16, device="cuda:0")
    return x[offset:].view(1, 1, GRID[1] * GRID[2], 64)


def calls():
    q, k, v, o = (bf16() for _ in range(4))
    k_odd, v_odd = bf16(1), bf16(1)
    n_tiles = 6
    counts, lists = (torch.empty(shape, dtype=torch.int32, device="cuda:0") for shape in ((1, n_tiles), (1, n_tiles, n_tiles)))
    return {
        "permute": lambda: sta.sta_tile_permute(q, o, GRID, TILE),
        "untile": lambda: sta.sta_untile(q, o, GRID, TILE),
        "forward": lambda: sta.sta_forward(q, k, v, o, GRID, TILE, WINDOWS),
        "forward, K and V at odd addresses": lambda: sta.sta_forward(q, k_odd, v_odd, o, GRID, TILE, WINDOWS),
        "general forward": lambda: sta.sta_forward_general(q, k, v, o, GRID, TILE, sta.STA_MASK_STA, WINDOWS),
        "key tiles": lambda: sta.sta_dump_key_tiles(1, GRID, TILE, WINDOWS, counts, lists),
    }


@pytest.mark.parametrize("name", ["permute", "untile", "forward", "forward, K and V at odd addresses", "general forward", "key tiles"])
def test_an_older_error_is_not_reported(name):
    call = calls()[name]
    call()                                              # with no error left: everything of a first call is done
    torch.cuda.synchronize()
    hip = sta.load_library()                            # (the runtime that it is linked with)
    hip.hipGetLastError()
    try:
        assert hip.hipSetDevice(ctypes.c_int(4096)) != 0    # no such device: refused on the host
        call()                                          # raises where the entry point returns an error
    finally:
        hip.hipGetLastError()
    torch.cuda.synchronize()
