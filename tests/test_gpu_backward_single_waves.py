"""Gradient launches of four walk groups of one wave beyond one workgroup per CU (dQ) or beyond short walks (dK/dV): which launches take
them (counted on 256 CUs, no GPU needed) and GPU parity at the edges of the rules."""
import numpy as np
import pytest

import synth_inputs as syn
from tests.launch_shapes import launches
from tests.test_gpu_backward import assert_grad_parity, gpu_backward, oracle_backward

# name, head dimensions, grid, tile, batch, heads, per-head windows repeated over the heads
SINGLE = [
    ("p384-768", (64,), (12, 32, 32), (6, 8, 8), 1, 2, [(1, 1, 3), (1, 1, 1)]),           # 768 waves; 36 sub-blocks and 12
    ("p384-432", (128,), (12, 24, 24), (6, 8, 8), 1, 2, [(1, 2, 3), (1, 1, 1)]),          # 432; 108 and 12
    ("p64-512", (64, 128), (1, 64, 64), (1, 8, 8), 2, 2, [(1, 8, 8), (1, 1, 1)]),         # 512; 128 and 2
    ("p192-1020", (64, 128), (3, 16, 40), (3, 8, 8), 1, 17, [(1, 1, 5)]),                 # 1020; 30
    ("p96-512", (64, 128), (2, 12, 16), (2, 6, 8), 21, 2, [(1, 2, 2), (1, 2, 2)]),        # 504 of at most 512; 12
    ("p96-504", (64, 128), (4, 18, 32), (2, 6, 8), 1, 7, [(1, 3, 3)]),                    # 504; 27
    ("p96-360", (128,), (4, 18, 40), (2, 6, 8), 1, 4, [(1, 3, 3), (1, 1, 1)]),            # 360; 27 and 3
    ("p160-480", (64, 128), (5, 24, 16), (5, 8, 4), 2, 4, [(1, 1, 3), (1, 1, 3)]),        # 480; 15
    ("p32-1024", (64,), (1, 32, 64), (1, 4, 8), 2, 8, [(1, 5, 7), (1, 1, 1)]),            # 1024; 35 and 1
]
TAKES = {("p96-512", 128): False}
OTHERS = [
    (64, (1, 64, 72), (1, 8, 8), 8, [(1, 8, 9)], "dq<64,2,2,1>"),          # 1152 waves
    (64, (1, 64, 64), (1, 8, 8), 4, [(1, 3, 3)], "dq<64,2,2,1>"),          # 18 sub-blocks
    (128, (1, 64, 64), (1, 8, 8), 4, [(1, 5, 5)], "dq<128,2,2,1>"),        # 50
    (128, (3, 16, 40), (3, 8, 8), 12, [(1, 1, 5)], "dq<128,3,2,1>"),       # 720 waves
    (128, (3, 16, 40), (3, 8, 8), 16, [(1, 1, 5), (1, 1, 1)], "dq<128,3,2,1>"),
    (64, (1, 32, 64), (1, 4, 8), 10, [(1, 3, 5)], "dq<64,1,1,1>"),         # 640 waves of 15
]
# dK/dV: name, head dimension, grid, tile, heads, windows
KEYS = [
    ("dkv-p384-720", 64, (6, 32, 40), (6, 8, 8), 3, [(1, 3, 3), (1, 1, 1)]),             # 720 waves; 108 sub-blocks, up to 192 of a key tile
    ("dkv-p256-768", 64, (8, 16, 24), (4, 8, 8), 8, [(1, 2, 3)]),                        # 768; 48
    ("dkv-p128-448", 128, (2, 64, 56), (2, 8, 8), 2, [(1, 5, 7), (1, 1, 1)]),            # 448; 140, up to 224
    ("dkv-p160-640", 64, (5, 32, 32), (5, 8, 4), 4, [(1, 1, 7)]),                        # 640; 35
    ("dkv-p224-756", 128, (21, 32, 12), (7, 8, 4), 3, [(1, 2, 2)]),                      # 756; 63
    ("dkv-p160-1000", 64, (5, 40, 32), (5, 8, 4), 5, [(1, 4, 1), (1, 2, 6)]),            # 1000; 105 and 25
]
OTHER_KEYS = [
    (64, (6, 64, 16), (6, 8, 8), 3, [(1, 2, 1)], "dkv<64,2,2,1,1>"),                     # 576 waves of 36
    (128, (6, 32, 40), (2, 8, 8), 2, [(3, 4, 4)], "dkv<128,2,2,1,1>"),                   # 480 of 240, all equal
    (128, (8, 48, 48), (4, 8, 8), 1, [(1, 4, 3)], "dkv<128,2,2,1,1>"),                   # 576 of 120
    (128, (5, 64, 8), (5, 8, 4), 8, [(1, 8, 1)], "dkv_pair<1,1,1>"),                     # 640 of 40
    (64, (10, 16, 20), (5, 8, 4), 8, [(2, 2, 5)], "dkv<64,1,2,1,1>"),                    # 800 of 100, all equal
    (128, (5, 40, 8), (5, 8, 4), 14, [(1, 5, 2)], "dkv_pair<1,1,1>"),                    # 700 of 50, all equal
    (128, (4, 16, 64), (2, 8, 8), 4, [(1, 4, 3)], "dkv<128,2,2,1,1>"),                   # 512 of 48, up to 64
]


def test_dkv_single_waves_where_walks_are_long_or_uneven():
    for name, D, grid, tile, H, windows in KEYS:
        line = launches(1, H, D, grid, tile, windows, gradients=True)[1]
        assert line.startswith("dkv<%d,1,4,1,1> items" % D), (name, line)
    for D, grid, tile, H, windows, want in OTHER_KEYS:
        assert launches(1, H, D, grid, tile, windows, gradients=True)[1].startswith(want + " "), (D, grid, H, windows)


def test_single_waves_where_walks_are_long():
    for name, dims, grid, tile, B, H, windows in SINGLE:
        for D in dims:
            line = launches(B, H, D, grid, tile, windows, gradients=True)[0]
            # two buffers for each operand as long as every workgroup is resident with them: one to a CU, two at head dimension 64
            kernel = "dq" if B * H * np.prod(grid) // 32 <= (512 if D == 64 else 256) else "dq_one_buffer"
            assert line.startswith("%s<%d,1,4,1> items" % (kernel, D)) == TAKES.get((name, D), True), (name, line)
    for D, grid, tile, H, windows, want in OTHERS:
        assert launches(1, H, D, grid, tile, windows, gradients=True)[0].startswith(want + " "), (D, grid, H, windows)


# dQ, one wave alone, one buffer for each operand: where the long walks are more than are resident with two, or all walks 1.25 times an even share
ALONE = [
    ("p32-2368", 64, (1, 32, 64), (1, 4, 8), 1, 37, [(1, 3, 5)]),                        # 2368 waves, 2304 resident; 15 sub-blocks
    ("p32-4672", 64, (1, 32, 64), (1, 4, 8), 1, 73, [(1, 3, 5), (1, 1, 1)]),             # 2368 of 15 and 2304 of 1
    ("p160-1050", 128, (5, 16, 28), (5, 8, 4), 1, 15, [(1, 1, 5)]),                      # 1050, 1024 resident; 25
    ("p160-2310", 128, (5, 16, 28), (5, 8, 4), 1, 33, [(1, 1, 5), (1, 2, 1), (1, 2, 1), (1, 2, 1)]),     # 630 of 25 and 1680 of 10
]
# ... and with two
TWO_BUFFERS = [
    (64, (1, 32, 64), (1, 4, 8), 64 + 1, [(1, 3, 5)]),                                   # 4160: the second round with one, and the end of two with two
    (128, (7, 72, 20), (7, 8, 4), 4, [(1, 2, 5), (1, 1, 1)]),                            # 1260, half of them of 7 sub-blocks beside 105
    (128, (1, 36, 64), (1, 4, 8), 24, [(1, 9, 7), (1, 3, 1)]),                           # 1728 of 63 and 3
]


def test_one_buffer_where_a_wave_alone_fills_the_chip():
    for name, D, grid, tile, B, H, windows in ALONE:
        assert launches(B, H, D, grid, tile, windows, gradients=True)[0].startswith("dq_one_buffer<%d,1,1,1> items" % D), name
        assert launches(B, H - 1, D, grid, tile, windows, gradients=True)[0].startswith("dq<%d,1,1,1> items" % D), name
    for D, grid, tile, H, windows in TWO_BUFFERS:
        assert launches(1, H, D, grid, tile, windows, gradients=True)[0].startswith("dq<%d,1,1,1> items" % D), (D, grid, H)


@pytest.mark.gpu
@pytest.mark.parametrize("name,D,grid,tile,B,H,windows", [(n, D, *rest) for n, dims, *rest in SINGLE for D in dims]
                         + [(n, D, grid, tile, 1, H, windows) for n, D, grid, tile, H, windows in KEYS] + ALONE,
                         ids=["%s-d%d" % (s[0], D) for s in SINGLE for D in s[1]] + ["%s-d%d" % s[:2] for s in KEYS + ALONE])
def test_gradients_of_single_waves_match_the_oracle(name, D, grid, tile, B, H, windows):
    w = syn.custom("bwd-single-" + name, B, H, D, grid, tile, [windows[h % len(windows)] for h in range(H)], "bf16", seed=2020)
    q, k, v = syn.make_qkv(w)
    g = syn.make_dout(w)
    (dq, dk, dv), _ = gpu_backward(w, q, k, v, g)
    for b, h in {(0, 0), (B - 1, H - 1)}:
        rq, rk, rv = oracle_backward(w, q, k, v, g, b, h)
        for label, got, ref in (("dQ", dq, rq), ("dK", dk, rk), ("dV", dv, rv)):
            assert_grad_parity(got[b, h].float().numpy(), ref, "%s D%d %s b%d h%d" % (name, D, label, b, h))
