"""GPU parity of every shape of the forward kernels that small and middle-sized launches take, on ordinary inputs, on keys masked
at the start of a walk and on scores that grow along it (both of which make items run again): waves on their own (a key share each,
32 or 64 queries per wave) and key groups that share LDS stages.  Counts of waves are on 256 CUs; every other head holds the same
data, so that the oracle looks at two.  (test_launch_rules.py says which kernel each of them runs.)"""
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

LAUNCHES = [
    # name, head dimension, grid, tile, heads, window; waves of 32 queries, units of 32 keys
    ("own-p64-32q-8", 64, (1, 40, 56), (1, 8, 8), 2, (1, 5, 7)),              # 140, 70
    ("own-p64-32q-4", 64, (1, 40, 56), (1, 8, 8), 6, (1, 3, 3)),              # 420, 18
    ("own-p64-64q-8", 64, (1, 40, 56), (1, 8, 8), 6, (1, 5, 5)),              # 420, 50
    ("own-p64-64q-4", 64, (1, 40, 56), (1, 8, 8), 10, (1, 3, 7)),             # 700, 42
    ("own-p192-64q-4", 64, (3, 24, 40), (3, 8, 8), 8, (1, 3, 5)),             # 720, 90
    ("own-p384-64q-8", 64, (6, 16, 24), (6, 8, 8), 4, (1, 2, 3)),             # 288, 72
    ("own-p96-4", 64, (4, 18, 40), (2, 6, 8), 20, (1, 3, 3)),                 # 1800, 27
    ("own-p32-4", 64, (1, 16, 48), (1, 4, 8), 30, (1, 3, 6)),                 # 720, 18
    ("own-p160-8", 64, (5, 8, 12), (5, 8, 4), 2, (1, 1, 4)),                  # 30, 15
    ("own-p384-d128-8", 128, (6, 16, 24), (6, 8, 8), 2, (1, 2, 2)),           # 144, 72
    ("own-p128-d128-4", 128, (4, 24, 24), (2, 8, 8), 2, (1, 3, 3)),           # 144, 36
    ("own-p64-d128-4", 128, (1, 40, 56), (1, 8, 8), 6, (1, 3, 3)),            # 420, 18
    ("own-p192-d128-4", 128, (3, 24, 40), (3, 8, 8), 8, (1, 3, 3)),           # 720, 54
    ("own-p32-d128-4", 128, (1, 16, 48), (1, 4, 8), 20, (1, 3, 5)),           # 480, 15
    ("shared-p64-two", 64, (1, 40, 56), (1, 8, 8), 16, (1, 3, 3)),            # 1120, 18
    ("shared-p64-one", 64, (1, 40, 56), (1, 8, 8), 30, (1, 3, 3)),            # 2100
    ("shared-p192-two", 64, (3, 24, 40), (3, 8, 8), 16, (1, 3, 3)),           # 1440, 54
    ("shared-p192-three-two", 64, (3, 24, 40), (3, 8, 8), 7, (1, 1, 3)),      # 630, 18
    ("shared-p192-three-one", 64, (3, 24, 40), (3, 8, 8), 24, (1, 3, 3)),     # 2160, 54
    ("shared-p96", 64, (4, 18, 40), (2, 6, 8), 24, (1, 3, 3)),                # 2160, 27
    ("shared-p32-two", 64, (1, 16, 48), (1, 4, 8), 34, (1, 3, 6)),            # 816, 18
    ("shared-p32-one", 64, (1, 16, 48), (1, 4, 8), 34, (1, 3, 3)),            # 816, 9
    ("shared-p384-d128-four", 128, (6, 16, 24), (6, 8, 8), 6, (1, 2, 2)),     # 432, 72
    ("shared-p384-d128-two", 128, (6, 16, 24), (6, 8, 8), 10, (1, 2, 3)),     # 720, 72
    ("shared-p384-d128-one", 128, (6, 16, 24), (6, 8, 8), 16, (1, 2, 2)),     # 1152
    ("shared-p64-d128-two", 128, (1, 40, 56), (1, 8, 8), 10, (1, 3, 3)),      # 700, 18
    ("shared-p64-d128-one", 128, (1, 40, 56), (1, 8, 8), 16, (1, 3, 3)),      # 1120
    ("shared-p96-d128-two", 128, (4, 18, 40), (2, 6, 8), 8, (1, 3, 3)),       # 720, 27
    ("shared-p96-d128-one", 128, (4, 18, 40), (2, 6, 8), 14, (1, 3, 3)),      # 1260
    ("shared-p32-d128", 128, (1, 16, 48), (1, 4, 8), 30, (1, 3, 5)),          # 720, 15
    # 48 queries shared by twelve waves
    ("own-p384-48q-12", 64, (6, 24, 24), (6, 8, 8), 3, (1, 3, 3)),            # 324, 108
    ("own-p192-48q-12", 64, (3, 24, 40), (3, 8, 8), 4, (1, 3, 3)),            # 360, 54
    # one LDS stage of V: with two groups, one, one wave of queries; tiles of many units; short walks
    ("one-v-p64-d128-two", 128, (1, 40, 56), (1, 8, 8), 18, (1, 3, 3)),       # 1260, 18
    ("one-v-p64-d128-one", 128, (1, 40, 56), (1, 8, 8), 34, (1, 3, 3)),       # 2380
    ("one-v-p320-d128", 128, (5, 24, 40), (5, 8, 8), 16, (1, 2, 3)),          # 2400, 90
    ("one-v-p64-d128-short", 128, (1, 40, 56), (1, 8, 8), 34, (1, 1, 3)),     # 2380, 6
    ("one-v-p32-d128", 128, (1, 16, 48), (1, 4, 8), 46, (1, 3, 5)),           # 1104, 15
    ("one-v-p32-d128-short", 128, (1, 16, 48), (1, 4, 8), 46, (1, 1, 3)),     # 1104, 3
]


def inputs(w, kind):
    if kind != "grow":
        return masked_inputs(w, float(kind[6:])) if kind.startswith("masked") else syn.make_qkv(w)
    q, k, v = syn.make_qkv(w)
    ramp = torch.empty(w.N)
    ramp[torch.from_numpy(orc.tile_order(w.grid, w.tile))] = torch.linspace(0.02, 14.0, w.N)        # along the tiled sequence
    return (q.float() * 2.0).to(torch.bfloat16), (k.float() * ramp[None, None, :, None]).to(torch.bfloat16), v


@pytest.mark.parametrize("kind", ["plain", "masked1", "masked4", "grow"])
@pytest.mark.parametrize("name,D,grid,tile,heads,window", LAUNCHES, ids=[s[0] for s in LAUNCHES])
def test_launches_match_the_oracle(name, D, grid, tile, heads, window, kind):
    w = syn.custom("launch-" + name, 1, 2, D, grid, tile, [window] * 2, "bf16", seed=616)
    q, k, v = inputs(w, kind)
    order = torch.from_numpy(orc.tile_order(w.grid, w.tile))
    index = torch.arange(heads) % 2
    qt, kt, vt = (x[:, index][:, :, order].contiguous().to(DEV) for x in (q, k, v))
    o = torch.full_like(qt, float("nan"))
    lse = torch.full(qt.shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    sta.sta_forward_lse(qt, kt, vt, o, lse, w.grid, w.tile, [window] * heads)
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), o[:, index].view(torch.int16)) and torch.equal(lse, lse[:, index])
    for h in range(2):
        ref, ref_lse = orc.attention(q[0, h].float().numpy(), k[0, h].float().numpy(), v[0, h].float().numpy(), w.grid, w.tile,
                                     orc.window_tiles_to_tokens(window, w.tile), return_lse=True)
        gu.assert_parity(o[0, h].float().cpu().numpy(), ref[order.numpy()], "%s %s h%d" % (name, kind, h))
        # bf16-rounded probabilities are summed, 2^-8 relative each at most, which is what is left where one key has nearly all the
        # weight (growing scores); the offset and the scores are fp32 numbers of the size of the result: 2^-22 of it
        want = ref_lse[order.numpy()]
        assert (np.abs(lse[0, h].cpu().numpy() - want) <= 2.0 ** -8 + 2.0 ** -22 * np.abs(want)).all()


@pytest.mark.parametrize("name,grid,tile,heads", [("one-v-p64-d128", (1, 40, 56), (1, 8, 8), 34), ("one-v-p32-d128", (1, 16, 48), (1, 4, 8), 46)])
def test_walks_of_one_tile_in_one_stage_of_v(name, grid, tile, heads):
    test_launches_match_the_oracle(name + "-one-tile", 128, grid, tile, heads, (1, 1, 1), "plain")


@pytest.mark.parametrize("D,grid,tile,window,groups", [(64, (1, 32, 32), (1, 8, 8), (1, 4, 4), 8), (128, (2, 32, 32), (2, 8, 8), (1, 4, 4), 8),
                                                       (64, (1, 16, 48), (1, 8, 8), (1, 2, 3), 4), (64, (6, 32, 48), (3, 8, 8), (2, 4, 6), 12)])
def test_accumulators_that_only_their_merge_would_take_out_of_range(D, grid, tile, window, groups):
    """Up to twelve key shares, each a quarter of the range's end with the offset of its first keys: the first 32 keys of every
    tile are zero, the others exceed them by 2^79 or so, under V = 2^b everywhere."""
    w = syn.custom("merge-range-8", 1, 1, D, grid, tile, [window], "bf16", seed=1)
    unit_of_key = torch.arange(w.N) % w.P // 32
    hot = (unit_of_key > 0).to(torch.float32) * (4.875 if D == 128 else 6.875)
    exponent = float(hot.max()) * D * D ** -0.5 * 1.4426950408889634 + np.log2((unit_of_key > 0).sum().item() / groups)
    for end in (127.97, 125.5):                                     # a share just below 2^128; the sum of all just beyond it
        b = int(np.floor(end - exponent))
        k = hot[None, None, :, None].expand(1, 1, w.N, D).to(torch.bfloat16).to(DEV)
        q = torch.ones_like(k)
        v = torch.full_like(k, 2.0 ** b)
        o, lse = torch.empty_like(k), torch.empty((1, 1, w.N), dtype=torch.float32, device=DEV)
        sta.sta_forward_lse(q, k.contiguous(), v, o, lse, w.grid, w.tile, w.window_tiles)
        got = o.float().cpu() * 2.0 ** -b
        assert torch.isfinite(got).all() and (got - 1).abs().max().item() <= 2.0 ** -7
