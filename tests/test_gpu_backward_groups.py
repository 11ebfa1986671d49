"""GPU parity of the gradient kernels at the edges of their shapes: every number of waves per workgroup, one and more walk
groups, shares of the walk that do not divide evenly or hold nothing."""
import numpy as np
import pytest
import torch

import synth_inputs as syn
from oracle import sta_oracle as orc
from tests.launch_shapes import launches
from tests.test_gpu_backward import assert_grad_parity, gpu_backward, oracle_backward

pytestmark = pytest.mark.gpu

# (grid, tile, batch, heads, per-head windows repeated over the heads).  Walk groups need 16 sub-blocks of 32 tokens in the widest
# head; the launches are small enough to fit the chip in groups except where many heads are asked for.
SHAPES = [
    ("p32", (1, 16, 48), (1, 4, 8), 1, 2, [(1, 3, 5), (1, 1, 1)]),
    ("p64-one", (1, 40, 56), (1, 8, 8), 1, 2, [(1, 1, 7), (1, 1, 1)]),          # 14 and 2 sub-blocks: one group
    ("p64-groups", (1, 40, 56), (1, 8, 8), 2, 2, [(1, 3, 3), (1, 2, 3)]),       # 18
    ("p64-empty", (1, 40, 56), (1, 8, 8), 1, 2, [(1, 5, 7), (1, 1, 1)]),        # 70 and 2: a group without a sub-block
    ("p96-one", (4, 18, 40), (2, 6, 8), 1, 2, [(1, 1, 5), (1, 1, 1)]),          # 15 and 3
    ("p96-two", (4, 18, 40), (2, 6, 8), 1, 2, [(2, 3, 5), (1, 1, 1)]),          # 90 and 3
    ("p128-one", (4, 24, 24), (2, 8, 8), 1, 2, [(1, 1, 3), (1, 1, 1)]),         # 12 and 4
    ("p128-groups", (4, 24, 24), (2, 8, 8), 1, 2, [(2, 1, 3), (1, 3, 1)]),      # 24 and 12
    ("p160", (5, 8, 12), (5, 8, 4), 1, 2, [(1, 1, 3), (1, 1, 1)]),
    ("p192", (3, 8, 216), (3, 8, 8), 1, 8, [(1, 1, 1), (1, 1, 2)]),             # three waves in dQ, two pairs in dK/dV
    # equal windows: rows of tiles over all heads, on the 96-token tiles the longest boxes first
    ("rows-p64", (1, 72, 40), (1, 8, 8), 2, 3, [(1, 5, 3)]),
    ("rows-p128", (10, 16, 40), (2, 8, 8), 1, 2, [(3, 1, 4)]),
    ("rows-p96", (6, 30, 8), (2, 6, 8), 1, 2, [(1, 3, 1)]),
    ("p384-groups", (6, 16, 24), (6, 8, 8), 1, 2, [(1, 2, 2), (1, 1, 1)]),      # 72 and 12
]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("name,grid,tile,B,H,windows", SHAPES, ids=[s[0] for s in SHAPES])
def test_gradient_kernel_shapes_match_the_oracle(name, grid, tile, B, H, windows, D):
    w = syn.custom("bwd-" + name, B, H, D, grid, tile, [windows[h % len(windows)] for h in range(H)], "bf16", seed=1212)
    q, k, v = syn.make_qkv(w)
    g = syn.make_dout(w)
    (dq, dk, dv), _ = gpu_backward(w, q, k, v, g)
    for b in range(B):
        for h in range(min(H, 2)):
            rq, rk, rv = oracle_backward(w, q, k, v, g, b, h)
            for label, got, ref in (("dQ", dq, rq), ("dK", dk, rk), ("dV", dv, rv)):
                assert_grad_parity(got[b, h].float().numpy(), ref, "%s D%d %s b%d h%d" % (name, D, label, b, h))


# Launches of 384-token tiles with at least 205 column blocks of 192 keys, whole heads: beyond what six pairs take in one round on
# 256 CUs (four waves, two groups of two), and in one round of them.
SIX_PAIRS = [
    # equal windows and two rounds: the rows of all heads in turn
    ("six-rows", (12, 32, 32), 8, [(1, 3, 1)]),
    # head after head: unequal windows, and equal ones in one round whose walks over the queries differ
    ("six-mixed", (6, 8, 216), 4, [(1, 1, 1), (1, 1, 2)]),
    ("six-one-round", (6, 8, 216), 4, [(1, 1, 4)]),
    # six pairs: one round, equal walks
    ("six-full", (6, 24, 24), 14, [(1, 1, 3), (1, 3, 1)]),
]


@pytest.mark.parametrize("name,grid,H,windows", SIX_PAIRS, ids=[s[0] for s in SIX_PAIRS])
def test_six_pair_gradients_match_the_oracle(name, grid, H, windows):
    w = syn.custom("bwd-" + name, 1, H, 128, grid, (6, 8, 8), [windows[h % len(windows)] for h in range(H)], "bf16", seed=1313)
    q, k, v = syn.make_qkv(w)
    g = syn.make_dout(w)
    (dq, dk, dv), _ = gpu_backward(w, q, k, v, g)
    for h in (0, H - 1):
        rq, rk, rv = oracle_backward(w, q, k, v, g, 0, h)
        for label, got, ref in (("dQ", dq, rq), ("dK", dk, rk), ("dV", dv, rv)):
            assert_grad_parity(got[0, h].float().numpy(), ref, "%s %s h%d" % (name, label, h))


def test_six_pair_kept_set_read_from_dv():
    """The transposed key-tile sets where every head has its own window (which no six pairs take): with Q = 0 a kept key has the
    probability 1 / (kept keys), so with dO one-hot in the query's tile dV_j[c] is 1 / (kept tiles of c) where c keeps j, else 0."""
    windows = [(1, 3, 2), (2, 1, 3), (1, 1, 1), (3, 3, 1), (2, 2, 4)]
    w = syn.custom("bwd-six-kept", 1, len(windows), 128, (12, 24, 32), (6, 8, 8), windows, "bf16", seed=1)      # 240 blocks
    z = torch.zeros((1, w.H, w.N, 128), dtype=torch.bfloat16)
    g = torch.zeros_like(z)
    order = orc.tile_order(w.grid, w.tile)
    tile_of_raster = np.empty(w.N, dtype=np.int64)
    tile_of_raster[order] = np.repeat(np.arange(w.n_tiles), w.P)
    g[0, :, torch.arange(w.N), torch.from_numpy(tile_of_raster)] = 1.0
    (_, _, dv), _ = gpu_backward(w, z, z.clone(), torch.ones_like(z), g)
    for h, window in enumerate(windows):
        counts, lists = orc.key_tiles(w.grid, w.tile, orc.window_tiles_to_tokens(window, w.tile))
        got = dv[0, h].float().numpy()[order].reshape(w.n_tiles, w.P, 128)
        for j in range(w.n_tiles):
            want = np.array([1.0 / counts[c] if j in lists[c][:counts[c]] else 0.0 for c in range(w.n_tiles)])
            assert np.allclose(got[j][:, :w.n_tiles], want[None, :], rtol=2.0 ** -7, atol=0), (h, j)
        assert (got[:, :, w.n_tiles:] == 0).all()


def test_kept_set_of_six_pairs_read_from_dv():
    """The same in a launch that six pairs take: one round, every head a window of three tiles along one of two axes."""
    windows = [(1, 1, 3), (1, 3, 1)] * 6
    assert launches(1, 12, 128, (6, 24, 24), (6, 8, 8), windows, gradients=True)[1].startswith("dkv_pair<6,1,1> items 216,")
    w = syn.custom("bwd-six-kept-round", 1, 12, 128, (6, 24, 24), (6, 8, 8), windows, "bf16", seed=1)
    z = torch.zeros((1, w.H, w.N, 128), dtype=torch.bfloat16)
    g = torch.zeros_like(z)
    order = orc.tile_order(w.grid, w.tile)
    tile_of_raster = np.empty(w.N, dtype=np.int64)
    tile_of_raster[order] = np.repeat(np.arange(w.n_tiles), w.P)
    g[0, :, torch.arange(w.N), torch.from_numpy(tile_of_raster)] = 1.0
    (_, _, dv), _ = gpu_backward(w, z, z.clone(), torch.ones_like(z), g)
    for h, window in enumerate(windows):
        counts, lists = orc.key_tiles(w.grid, w.tile, orc.window_tiles_to_tokens(window, w.tile))
        got = dv[0, h].float().numpy()[order].reshape(w.n_tiles, w.P, 128)
        for j in range(w.n_tiles):
            want = np.array([1.0 / counts[c] if j in lists[c][:counts[c]] else 0.0 for c in range(w.n_tiles)])
            assert np.allclose(got[j][:, :w.n_tiles], want[None, :], rtol=2.0 ** -7, atol=0), (h, j)
        assert (got[:, :, w.n_tiles:] == 0).all()
