"""GPU parity of the kernels that serve the large launches at head dimension 128 (tiles of 128 tokens' multiples, more than 1280
waves of queries): 12 and 4 waves per workgroup, whole items and, with a workspace, items cut into parts along the keys.  Every
other head holds the same data, so that the launches are large and the oracle's work is small."""
import numpy as np
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


@pytest.mark.parametrize("name", LAUNCHES)
def test_items_are_done_again_where_scores_outgrow_the_first_offset(name):
    """Scores that grow along the walk from near zero by more than 2^100 in the exponent: the row sums leave the safe range.  In a
    split launch the parts restart where their share of the walk begins."""
    grid, tile, heads, workspace = LAUNCHES[name]
    w = syn.custom("large-outgrow", 1, 2, 128, grid, tile, [(1, 3, 3), (3, 3, 3)], "bf16", seed=84)
    q, k, v = syn.make_qkv(w)
    ramp = torch.empty(w.N)
    ramp[torch.from_numpy(orc.tile_order(w.grid, w.tile))] = torch.linspace(0.02, 14.0, w.N)
    k = (k.float() * ramp[None, None, :, None]).to(torch.bfloat16)
    q = (q.float() * 2.0).to(torch.bfloat16)
    check(w, q, k, v, run(w, q, k, v, heads, workspace), name)


@pytest.mark.parametrize("name", LAUNCHES)
def test_items_are_done_again_where_accumulators_leave_the_range(name):
    """One tile's keys exceed all others by 2^79 as a factor, V is scaled by 2^50: row sums stay below 2^96, accumulators pass
    2^128.  The result is 2^50 times that of the unscaled V."""
    grid, tile, heads, workspace = LAUNCHES[name]
    w = syn.custom("large-vhuge", 1, 2, 128, grid, tile, [(3, 3, 3), (1, 3, 3)], "bf16", seed=85)
    _, _, v = syn.make_qkv(w)
    order = torch.from_numpy(orc.tile_order(w.grid, w.tile))
    q = torch.ones((1, 2, w.N, 128), dtype=torch.bfloat16)
    k = torch.zeros_like(q)
    k[:, :, order[(w.n_tiles - 1) * w.P:], :] = 4.875
    out = run(w, q, k, (v.float() * 2.0 ** 50).to(torch.bfloat16), heads, workspace)
    check(w, q, k, v, out.float() * 2.0 ** -50, name)


@pytest.mark.parametrize("name", LAUNCHES)
def test_all_scores_far_below_zero(name):
    """The first offset has to move down from zero."""
    grid, tile, heads, workspace = LAUNCHES[name]
    w = syn.custom("large-negative", 1, 2, 128, grid, tile, [(1, 1, 2), (1, 2, 2)], "bf16", seed=83)
    q, k, v = syn.make_qkv(w)
    q = (q.float().abs() * 3.0).to(torch.bfloat16)
    k = (-(k.float().abs()) * 3.0).to(torch.bfloat16)
    check(w, q, k, v, run(w, q, k, v, heads, workspace), name)


@pytest.mark.parametrize("name", LAUNCHES)
def test_outputs_repeat_bit_for_bit(name):
    grid, tile, heads, workspace = LAUNCHES[name]
    w = syn.custom("large-repro", 1, 2, 128, grid, tile, [(1, 2, 3), (3, 3, 3)], "bf16", seed=81)
    q, k, v = syn.make_qkv(w)
    first = run(w, q, k, v, heads, workspace)
    check(w, q, k, v, first, name)
    for _ in range(3):
        assert torch.equal(run(w, q, k, v, heads, workspace).view(torch.int16), first.view(torch.int16))


@pytest.mark.parametrize("grid,tile,heads,workspace", [
    ((12, 24, 32), (6, 8, 8), 16, False),          # 12 waves
    ((12, 24, 32), (6, 8, 8), 16, True),           # ... 384 items, the last 128 in two parts
    ((4, 24, 32), (2, 8, 8), 14, False),           # 4 waves
    ((4, 24, 32), (2, 8, 8), 14, True),            # ... 336 items in two parts each
], ids=["12-waves", "12-waves-parts", "4-waves", "4-waves-parts"])
def test_kept_set_read_from_the_output(grid, tile, heads, workspace):
    """Q = 0 and V one-hot in the key's tile: O[i, tau] = [tau kept] / kept tiles, every head with its own window."""
    choices = [(1, 3, 3), (2, 1, 4), (2, 3, 4), (1, 2, 4), (3, 9, 9)]
    windows = [choices[h % len(choices)] for h in range(heads)]
    w = syn.custom("large-onehot", 1, heads, 128, grid, tile, windows, "bf16", seed=11)
    q = torch.zeros((1, heads, w.N, 128), dtype=torch.bfloat16, device=DEV)
    k = torch.randn(q.shape, generator=torch.Generator(device=DEV).manual_seed(11), device=DEV).to(torch.bfloat16)
    v = torch.zeros_like(q)
    v[:, :, torch.arange(w.N, device=DEV), torch.arange(w.N, device=DEV) // w.P] = 1.0
    o = torch.full_like(q, float("nan"))
    ws = torch.zeros(sta.sta_workspace_bytes(1, heads, 128, grid, tile), dtype=torch.uint8, device=DEV) if workspace else None
    sta.sta_forward(q, k, v, o, grid, tile, windows, workspace=ws)
    if workspace:
        assert ws.any().item(), "no item was cut into parts"
    out = o[0].float().cpu().numpy().reshape(heads, w.n_tiles, w.P, 128)
    for h in range(heads):
        counts, lists = orc.key_tiles(grid, tile, orc.window_tiles_to_tokens(windows[h], tile))
        for qt in range(w.n_tiles):
            want = np.zeros(128)
            want[lists[qt, :counts[qt]]] = 1.0 / counts[qt]
            assert np.allclose(out[h, qt], want[None, :], rtol=2.0 ** -7, atol=0), (h, qt)


@pytest.mark.parametrize("name", [n for n, launch in LAUNCHES.items() if not launch[3]])
def test_log_denominators(name):
    grid, tile, heads, _ = LAUNCHES[name]
    w = syn.custom("large-lse", 1, 2, 128, grid, tile, [(1, 2, 3), (3, 3, 3)], "bf16", seed=82)
    q, k, v = syn.make_qkv(w)
    order = orc.tile_order(w.grid, w.tile)
    index = torch.arange(heads) % 2
    qt, kt, vt = (x[:, index][:, :, torch.from_numpy(order)].contiguous().to(DEV) for x in (q, k, v))
    o = torch.full_like(qt, float("nan"))
    lse = torch.full(qt.shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    sta.sta_forward_lse(qt, kt, vt, o, lse, w.grid, w.tile, [w.window_tiles[h % 2] for h in range(heads)])
    check(w, q, k, v, o, name)
    for h in range(2):
        _, ref = orc.attention(q[0, h].float().numpy(), k[0, h].float().numpy(), v[0, h].float().numpy(), w.grid, w.tile,
                               orc.window_tiles_to_tokens(w.window_tiles[h], w.tile), return_lse=True)
        # bf16-rounded probabilities are summed: 2^-9 relative each, so below 2^-9 = 2e-3 in the log
        for head in (h, heads - heads % 2 - 2 + h):
            assert np.abs(lse[0, head].cpu().numpy() - ref[order]).max() <= 2e-3
