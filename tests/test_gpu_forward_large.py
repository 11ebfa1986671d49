"""GPU parity of the kernels that serve the large launches at head dimension 128 (tiles of 128 tokens' multiples, more than 1280
waves of queries): 12 and 4 waves per workgroup, whole items and, with a workspace, items cut into parts along the keys.  Every
other head holds the same data, so that the launches are large and the oracle's work is small."""
import pytest
import torch

import paper_2502_04507_amd as sta
import synth_inputs as syn
from oracle import sta_oracle as orc
from tests import gpu_util as gu
from tests.test_gpu_masked_keys import masked_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (grid, tile, heads, workspace); 256 CUs hold 256 workgroups of 12 waves or 768 of 4
LAUNCHES = {
    "p384-4-waves": ((6, 16, 24), (6, 8, 8), 18, False),            # 108 items of 384 queries would leave a round half empty
    "p384-12-waves": ((6, 16, 24), (6, 8, 8), 30, False),           # 180 items
    "p384-12-waves-parts": ((6, 16, 24), (6, 8, 8), 18, True),      # 108 items in two parts each
    "p768-12-waves": ((6, 16, 32), (6, 8, 16), 30, False),          # 240 items, two per tile
    "p128-4-waves": ((4, 16, 16), (2, 8, 8), 41, False),            # 328 items of 128 queries
    "p128-4-waves-parts": ((4, 16, 16), (2, 8, 8), 41, True),       # ... in two parts each
}


def run(w, q, k, v, heads, workspace):
    """Tiled outputs of a launch over `heads` heads that hold the data of w's two heads in turn; with a workspace, asserts that
    partial results went through it."""
    order = torch.from_numpy(orc.tile_order(w.grid, w.tile))
    index = torch.arange(heads) % 2
    qt, kt, vt = (x[:, index][:, :, order].contiguous().to(DEV) for x in (q, k, v))
    o = torch.full_like(qt, float("nan"))
    ws = torch.zeros(sta.sta_workspace_bytes(1, heads, 128, w.grid, w.tile), dtype=torch.uint8, device=DEV) if workspace else None
    sta.sta_forward(qt, kt, vt, o, w.grid, w.tile, [w.window_tiles[h % 2] for h in range(heads)], workspace=ws)
    torch.cuda.synchronize()
    if workspace:
        assert ws.any().item(), "no item was cut into parts"
    return o


def check(w, q, k, v, out, label):
    """The first and the last two heads (other items of the launch) against the oracle."""
    order = orc.tile_order(w.grid, w.tile)
    refs = [gu.oracle_rows(w, q, k, v, 0, h, None)[order] for h in range(2)]
    for h in (0, 1, out.shape[1] - 2, out.shape[1] - 1):
        gu.assert_parity(out[0, h].float().cpu().numpy(), refs[h % 2], "%s head %d" % (label, h))


@pytest.mark.parametrize("channel", [1.0, 4.0])
@pytest.mark.parametrize("name", LAUNCHES)
def test_masked_keys_at_the_start_of_a_walk(name, channel):
    """Scores of the lowest fp32 number and of minus infinity, as in the tests of the key-group kernel."""
    grid, tile, heads, workspace = LAUNCHES[name]
    w = syn.custom("large-masked", 1, 2, 128, grid, tile, [(1, 2, 2), (3, 3, 3)], "bf16", seed=911)
    q, k, v = masked_inputs(w, channel)
    check(w, q, k, v, run(w, q, k, v, heads, workspace), name)
