"""GPU parity of the forward kernels whose workgroups share a walk between waves, at the edges of their shapes: shares of the walk
that do not divide evenly or hold nothing, tiles of every kind, accumulators that only their merge takes out of range, and the
log-denominators merged over the shares."""
import numpy as np
import pytest
import torch

import paper_2502_04507_amd as sta
import synth_inputs as syn
from oracle import sta_oracle as orc
from tests import gpu_util as gu
from tests.launch_shapes import launches

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# Launches of at most 256 waves, which the kernel of lone waves takes in four or eight key shares (p192-three-waves, 720 waves, in
# four): by the number of 32-key units of the widest head, which the names of the cases go by (one, two and four groups of the
# key-group kernel, further down in launches that it takes).  (grid, tile, per-head windows; units of each head)
SHAPES = [
    ("p32", (1, 16, 48), (1, 4, 8), [(1, 3, 5), (1, 1, 1)]),            # 15 and 1 units: shares without a unit
    ("p32-two", (1, 16, 48), (1, 4, 8), [(1, 3, 6), (1, 3, 5)]),        # 18 and 15: odd shares
    ("p96", (4, 18, 40), (2, 6, 8), [(1, 1, 5), (1, 1, 1)]),            # 15 and 3
    ("p96-two", (4, 18, 40), (2, 6, 8), [(1, 3, 3), (1, 1, 1)]),        # 27 and 3
    ("p96-four", (4, 18, 40), (2, 6, 8), [(2, 3, 5), (1, 1, 1)]),       # 90 and 3: shares without a unit
    ("p64", (1, 40, 56), (1, 8, 8), [(1, 1, 7), (1, 1, 1)]),            # 14 and 2
    ("p64-two", (1, 40, 56), (1, 8, 8), [(1, 3, 3), (1, 2, 3)]),        # 18
    ("p64-four", (1, 40, 56), (1, 8, 8), [(1, 5, 7), (1, 1, 1)]),       # 70 and 2: six of eight shares without a unit
    ("p128", (4, 24, 24), (2, 8, 8), [(1, 1, 3), (1, 1, 1)]),           # 12 and 4
    ("p128-two", (4, 24, 24), (2, 8, 8), [(2, 1, 3), (1, 3, 1)]),       # 24 and 12
    ("p160", (5, 8, 12), (5, 8, 4), [(1, 1, 3), (1, 1, 1)]),            # 15 and 5
    ("p192-two-waves", (3, 24, 40), (3, 8, 8), [(1, 3, 5), (1, 1, 1)]), # 90 and 6: shares without a unit
    ("p192-three-waves", (6, 24, 40), (3, 8, 8), [(1, 3, 3)] * 4),      # 54, 720 waves
    ("p384", (6, 16, 16), (6, 8, 8), [(1, 1, 1), (1, 1, 1)]),           # 12
    ("p384-four", (6, 16, 24), (6, 8, 8), [(1, 2, 2), (1, 1, 1)]),      # 72 and 12
]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("name,grid,tile,windows", SHAPES, ids=[s[0] for s in SHAPES])
def test_key_groups_match_the_oracle(name, grid, tile, windows, D):
    w = syn.custom(name, 1, len(windows), D, grid, tile, windows, "bf16", seed=5150)
    q, k, v = syn.make_qkv(w)
    order = torch.from_numpy(orc.tile_order(w.grid, w.tile))
    qt, kt, vt = (x[:, :, order].contiguous().to(DEV) for x in (q, k, v))
    o = torch.full_like(qt, float("nan"))
    lse = torch.full(qt.shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    sta.sta_forward_lse(qt, kt, vt, o, lse, w.grid, w.tile, w.window_tiles)
    again = torch.full_like(qt, float("nan"))
    sta.sta_forward(qt, kt, vt, again, w.grid, w.tile, w.window_tiles)
    torch.cuda.synchronize()
    assert torch.equal(again.view(torch.int16), o.view(torch.int16))
    order = order.numpy()
    for h in range(w.H):
        ref_o, ref_lse = orc.attention(q[0, h].float().numpy(), k[0, h].float().numpy(), v[0, h].float().numpy(), w.grid,
                                       w.tile, orc.window_tiles_to_tokens(w.window_tiles[h], w.tile), return_lse=True)
        gu.assert_parity(o[0, h].float().cpu().numpy(), ref_o[order], "%s D%d h%d" % (name, D, h))
        # bf16-rounded probabilities are summed: 2^-9 relative each, independent, so below 2^-9 = 2e-3 in the log
        assert np.abs(lse[0, h].cpu().numpy() - ref_lse[order]).max() <= 2e-3


@pytest.mark.parametrize("grid,tile,heads", [((6, 16, 24), (6, 8, 8), 18), ((6, 16, 24), (6, 8, 8), 30), ((4, 16, 16), (2, 8, 8), 41)],
                         ids=["p384-4-waves", "p384-12-waves", "p128-4-waves"])
def test_launches_beyond_the_key_groups_redo_items_whose_scores_grow(grid, tile, heads):
    """Head dimension 128 with more than 1280 waves of queries: 4- and 12-wave workgroups.  The scores grow along the walk by
    far more than fp32 sums can take with the first offset, so items are done again.  Every other head holds the same data."""
    w = syn.custom("outgrow-many", 1, 2, 128, grid, tile, [(1, 3, 3), (3, 3, 3)], "bf16", seed=84)
    q, k, v = syn.make_qkv(w)
    order = torch.from_numpy(orc.tile_order(w.grid, w.tile))
    ramp = torch.empty(w.N)
    ramp[order] = torch.linspace(0.02, 14.0, w.N)                       # along the tiled sequence
    k = (k.float() * ramp[None, None, :, None]).to(torch.bfloat16)
    q = (q.float() * 2.0).to(torch.bfloat16)
    index = torch.arange(heads) % 2
    qt, kt, vt = (x[:, index][:, :, order].contiguous().to(DEV) for x in (q, k, v))
    o = torch.full_like(qt, float("nan"))
    sta.sta_forward(qt, kt, vt, o, w.grid, w.tile, [w.window_tiles[h % 2] for h in range(heads)])
    torch.cuda.synchronize()
    for h in range(heads):
        assert torch.equal(o[:, h].view(torch.int16), o[:, h % 2].view(torch.int16)), h
    for h in range(2):
        ref = orc.attention(q[0, h].float().numpy(), k[0, h].float().numpy(), v[0, h].float().numpy(), w.grid, w.tile,
                            orc.window_tiles_to_tokens(w.window_tiles[h], w.tile))
        gu.assert_parity(o[0, h].float().cpu().numpy(), ref[order.numpy()], "outgrow-many h%d" % h)


@pytest.mark.parametrize("D,grid,tile,groups", [(64, (1, 32, 32), (1, 8, 8), 4), (64, (1, 16, 48), (1, 8, 8), 2),
                                                (128, (2, 32, 32), (2, 8, 8), 4), (128, (2, 16, 24), (2, 8, 8), 2)])
def test_merged_accumulators_of_key_groups_stay_in_range(D, grid, tile, groups):
    """In four or eight shares of lone waves: every one of `groups` accumulators ends just below 2^128 with the offset of its first keys, so their sum would not: the first 32
    keys of every tile are zero and the others exceed them by 2^79 (row sums stay below 2^96), under V = 2^b everywhere."""
    w = syn.custom("merge-range", 1, 1, D, grid, tile, [tuple(g // t for g, t in zip(grid, tile))], "bf16", seed=1)
    unit_of_key = torch.arange(w.N) % w.P // 32
    hot = (unit_of_key > 0).to(torch.float32) * (4.875 if D == 128 else 6.875)
    # log2 of a score factor: raw score x 1/sqrt(D) x log2(e); keys that count per group; then b for a sum in [2^127, 2^128)
    exponent = float(hot.max()) * D * D ** -0.5 * 1.4426950408889634 + np.log2((unit_of_key > 0).sum().item() / groups)
    b = int(np.floor(127.97 - exponent))
    assert 127 < exponent + b < 127.97
    k = hot[None, None, :, None].expand(1, 1, w.N, D).to(torch.bfloat16).to(DEV)
    q = torch.ones_like(k)
    v = torch.full_like(k, 2.0 ** b)
    o, lse = torch.empty_like(k), torch.empty((1, 1, w.N), dtype=torch.float32, device=DEV)
    sta.sta_forward_lse(q, k.contiguous(), v, o, lse, w.grid, w.tile, w.window_tiles)
    got = o.float().cpu() * 2.0 ** -b
    assert torch.isfinite(got).all()
    assert (got - 1).abs().max().item() <= 2.0 ** -7


@pytest.mark.parametrize("D,grid,tile,window,heads,kernel", [
    (64, (1, 32, 32), (1, 8, 8), (1, 4, 4), 40, "group<64,2,2,0,1>"), (64, (1, 16, 48), (1, 8, 8), (1, 2, 6), 30, "group<64,2,2,0,1>"),
    (64, (3, 24, 32), (3, 8, 8), (1, 1, 4), 8, "group<64,3,2,0,1>"), (128, (2, 32, 32), (2, 8, 8), (1, 4, 4), 6, "group<128,2,4,0,1>"),
    (128, (2, 16, 24), (2, 8, 8), (1, 2, 3), 20, "group<128,2,2,0,1>")])
def test_merged_accumulators_of_the_key_group_kernel_stay_in_range(D, grid, tile, window, heads, kernel):
    """The same in launches that the key-group kernel takes, two or four groups: a group's accumulators end just below 2^128, or just
    below a quarter of it, so that only their sum leaves the range.  Windows keep as many keys for every query, and every group
    begins with a tile."""
    assert launches(1, heads, D, grid, tile, [window])[0].startswith(kernel + " ")
    w = syn.custom("merge-range-many", 1, 1, D, grid, tile, [window], "bf16", seed=1)
    groups = int(kernel.split(",")[2])
    unit_of_key = torch.arange(w.N) % w.P // 32
    hot = (unit_of_key > 0).to(torch.float32) * (4.875 if D == 128 else 6.875)
    kept = np.prod([min(2 * (x // 2) + 1, g // t) for x, g, t in zip(window, grid, tile)]) * (w.P - 32)      # keys that count, per query
    exponent = float(hot.max()) * D * D ** -0.5 * 1.4426950408889634 + np.log2(kept / groups)
    for end in (127.97, 125.97):
        b = int(np.floor(end - exponent))
        k = hot[None, None, :, None].expand(1, heads, w.N, D).to(torch.bfloat16).to(DEV)
        q = torch.ones_like(k)
        v = torch.full_like(k, 2.0 ** b)
        o, lse = torch.empty_like(k), torch.empty((1, heads, w.N), dtype=torch.float32, device=DEV)
        sta.sta_forward_lse(q, k.contiguous(), v, o, lse, w.grid, w.tile, [window] * heads)
        got = o.float().cpu() * 2.0 ** -b
        assert torch.isfinite(got).all()
        assert (got - 1).abs().max().item() <= 2.0 ** -7


@pytest.mark.parametrize("name,D,grid,tile,heads,windows,kernel", [
    ("p32", 64, (1, 16, 48), (1, 4, 8), 40, [(1, 3, 6), (1, 1, 1)], "group<64,1,2,1,1>"),              # 960 waves; 18 units and 1
    ("p192", 64, (3, 24, 40), (3, 8, 8), 8, [(1, 1, 3), (1, 1, 1)], "group<64,3,2,0,1>"),              # 720; 18 and 6
    ("p64", 64, (1, 40, 56), (1, 8, 8), 16, [(1, 3, 3), (1, 1, 1)], "group<64,2,2,0,1>"),              # 1120; 18 and 2
    ("p64-d128", 128, (1, 40, 56), (1, 8, 8), 10, [(1, 3, 3), (1, 1, 1)], "group<128,2,2,1,1>"),       # 700; 18 and 2
    ("p96-d128", 128, (4, 18, 40), (2, 6, 8), 8, [(1, 3, 3), (1, 1, 1)], "group<128,3,2,1,1>"),        # 720; 27 and 3
    ("p128-d128", 128, (4, 24, 24), (2, 8, 8), 6, [(1, 3, 3), (1, 1, 1)], "group<128,2,4,0,1>"),       # 432; 36 and 4
])
def test_key_groups_with_little_or_nothing_to_walk(name, D, grid, tile, heads, windows, kernel):
    """Mixed windows in launches that the key-group kernel takes: on 32-token tiles the first group of a head that keeps one tile
    has no unit, elsewhere one or a few.  Every other head holds the same data; ordinary keys, keys masked at the start of a
    walk and scores that grow along it."""
    per_head = [windows[h % 2] for h in range(heads)]
    assert launches(1, heads, D, grid, tile, per_head)[0].startswith(kernel + " ")
    w = syn.custom("little-" + name, 1, 2, D, grid, tile, windows, "bf16", seed=717)
    order = torch.from_numpy(orc.tile_order(w.grid, w.tile))
    index = torch.arange(heads) % 2
    for kind in ("plain", "masked", "grow"):
        q, k, v = syn.make_qkv(w)
        if kind == "masked":                                            # every other tile's keys, not those of a window of one tile
            keys = torch.zeros(w.N, dtype=torch.bool)
            keys[order] = (torch.arange(w.n_tiles) % (w.grid[2] // w.tile[2]) % 2 == 0).repeat_interleave(w.P)
            q[..., 0] = 1.0
            k[..., 0] = 0.0
            k[0, 0, :, 0] = torch.where(keys, torch.finfo(torch.bfloat16).min, 0.0).to(torch.bfloat16)
        if kind == "grow":
            ramp = torch.empty(w.N)
            ramp[order] = torch.linspace(0.02, 14.0, w.N)
            q, k = (q.float() * 2.0).to(torch.bfloat16), (k.float() * ramp[None, None, :, None]).to(torch.bfloat16)
        qt, kt, vt = (x[:, index][:, :, order].contiguous().to(DEV) for x in (q, k, v))
        o = torch.full_like(qt, float("nan"))
        lse = torch.full(qt.shape[:3], float("nan"), dtype=torch.float32, device=DEV)
        sta.sta_forward_lse(qt, kt, vt, o, lse, w.grid, w.tile, per_head)
        torch.cuda.synchronize()
        assert torch.equal(o.view(torch.int16), o[:, index].view(torch.int16)) and torch.equal(lse, lse[:, index])
        for h in range(2):
            ref, ref_lse = orc.attention(q[0, h].float().numpy(), k[0, h].float().numpy(), v[0, h].float().numpy(), w.grid, w.tile,
                                         orc.window_tiles_to_tokens(windows[h], w.tile), return_lse=True)
            gu.assert_parity(o[0, h].float().cpu().numpy(), ref[order.numpy()], "%s %s h%d" % (name, kind, h))
            # the bound of test_gpu_forward_launches.py: rounded probabilities are summed, 2^-8 relative each at most, and the
            # offset and the scores are fp32 numbers of the size of the result
            want = ref_lse[order.numpy()]
            assert (np.abs(lse[0, h].cpu().numpy() - want) <= 2.0 ** -8 + 2.0 ** -22 * np.abs(want)).all()


@pytest.mark.parametrize("grid,tile,heads", [((6, 16, 24), (6, 8, 8), 30), ((4, 16, 16), (2, 8, 8), 66)], ids=["p384", "p128"])
def test_two_units_per_stage_redo_items_whose_scores_grow(grid, tile, heads):
    """Head dimension 64 with more than 2048 waves of queries and tiles of 128 tokens' multiples: no key groups, two units per
    stage.  The scores grow along the walk so that items are done again.  Every other head holds the same data."""
    w = syn.custom("outgrow-stages", 1, 2, 64, grid, tile, [(1, 3, 3), (3, 3, 3)], "bf16", seed=85)
    q, k, v = syn.make_qkv(w)
    order = torch.from_numpy(orc.tile_order(w.grid, w.tile))
    ramp = torch.empty(w.N)
    ramp[order] = torch.linspace(0.02, 14.0, w.N)                       # along the tiled sequence
    k = (k.float() * ramp[None, None, :, None]).to(torch.bfloat16)
    q = (q.float() * 2.0).to(torch.bfloat16)
    index = torch.arange(heads) % 2
    qt, kt, vt = (x[:, index][:, :, order].contiguous().to(DEV) for x in (q, k, v))
    o = torch.full_like(qt, float("nan"))
    sta.sta_forward(qt, kt, vt, o, w.grid, w.tile, [w.window_tiles[h % 2] for h in range(heads)])
    torch.cuda.synchronize()
    for h in range(heads):
        assert torch.equal(o[:, h].view(torch.int16), o[:, h % 2].view(torch.int16)), h
    for h in range(2):
        ref = orc.attention(q[0, h].float().numpy(), k[0, h].float().numpy(), v[0, h].float().numpy(), w.grid, w.tile,
                            orc.window_tiles_to_tokens(w.window_tiles[h], w.tile))
        gu.assert_parity(o[0, h].float().cpu().numpy(), ref[order.numpy()], "outgrow-stages h%d" % h)
