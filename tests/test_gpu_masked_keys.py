"""Keys that a caller masks through a channel: the queries hold a positive number there and the masked keys the lowest bf16
number, so their scores are the lowest fp32 numbers or minus infinity.  Where a walk (or a key group's share of one) begins
with such keys, the first exponent offset must neither swallow the scores that follow nor become infinite."""
import numpy as np
import pytest
import torch

import paper_2502_04507_amd as sta
import synth_inputs as syn
from oracle import sta_oracle as orc
from tests import gpu_util as gu
from tests.test_gpu_backward import assert_grad_parity, gpu_backward, oracle_backward

pytestmark = pytest.mark.gpu

# Key tiles with an even coordinate along the last axis are masked.  Every window holds tiles of both kinds; small launches, whose
# walks are shared by four or eight waves.  (name, grid, tile, per-head windows)
SHAPES = [
    ("p32", (1, 16, 48), (1, 4, 8), [(1, 3, 5), (1, 1, 2)]),
    ("p64", (1, 40, 56), (1, 8, 8), [(1, 1, 7), (1, 1, 3)]),
    ("p64-four", (1, 40, 56), (1, 8, 8), [(1, 5, 7), (1, 3, 3)]),
    ("p96-one", (4, 18, 40), (2, 6, 8), [(1, 1, 5), (1, 1, 3)]),
    ("p96-four", (4, 18, 40), (2, 6, 8), [(2, 3, 5), (1, 1, 3)]),
    ("p128", (4, 24, 24), (2, 8, 8), [(1, 1, 3), (1, 3, 2)]),
    ("p384-four", (6, 16, 24), (6, 8, 8), [(1, 2, 2), (1, 1, 3)]),
]
CASES = [(shape, D, channel) for shape in SHAPES for D in (64, 128) for channel in (1.0, 4.0)]


def masked_inputs(w, channel):
    q, k, v = syn.make_qkv(w)
    order = torch.from_numpy(orc.tile_order(w.grid, w.tile))
    n_w = w.grid[2] // w.tile[2]
    masked = torch.zeros(w.N, dtype=torch.bool)
    masked[order] = (torch.arange(w.n_tiles) % n_w % 2 == 0).repeat_interleave(w.P)
    q[..., 0] = channel
    k[..., 0] = torch.where(masked, torch.finfo(torch.bfloat16).min, 0.0).to(torch.bfloat16)
    return q, k, v


@pytest.mark.parametrize("shape,D,channel", CASES, ids=["%s-D%d-q%g" % (s[0], D, c) for s, D, c in CASES])
def test_masked_keys_at_the_start_of_a_walk(shape, D, channel):
    name, grid, tile, windows = shape
    w = syn.custom("masked-" + name, 1, len(windows), D, grid, tile, windows, "bf16", seed=909)
    q, k, v = masked_inputs(w, channel)
    for workspace in (False, True):
        out = gu.gpu_chain(w, q, k, v, workspace=workspace).float().numpy()
        for h in range(w.H):
            gu.assert_parity(out[0, h], gu.oracle_rows(w, q, k, v, 0, h, None), "%s D%d h%d" % (name, D, h))


@pytest.mark.parametrize("channel", [1.0, 4.0])
def test_gradients_with_masked_keys(channel):
    w = syn.custom("masked-bwd", 1, 1, 128, (4, 18, 40), (2, 6, 8), [(1, 3, 3)], "bf16", seed=910)
    q, k, v = masked_inputs(w, channel)
    g = syn.make_dout(w)
    grads, _ = gpu_backward(w, q, k, v, g)
    for label, got, ref in zip(("dQ", "dK", "dV"), grads, oracle_backward(w, q, k, v, g, 0, 0)):
        assert_grad_parity(got[0, 0].float().numpy(), ref, "masked %s" % label)
