"""Gradient launches of eight walk groups of one wave (at most one wave of columns per CU, walks of 40 sub-blocks or more, 44 at head dimension 128): which
launches take them (counted on 256 CUs, no GPU needed) and GPU parity at the edges of the rule, with shares that do not divide evenly
or hold nothing."""
import pytest

import synth_inputs as syn
from tests.launch_shapes import launches
from tests.test_gpu_backward import assert_grad_parity, gpu_backward, oracle_backward

# grid, tile, batch, heads, per-head windows repeated over the heads
EIGHT = [
    ("p64-256-waves", (1, 64, 64), (1, 8, 8), 1, 2, [(1, 4, 5), (1, 1, 1)]),        # walks of 50 and 2 (even windows round up to odd): empty groups
    ("p64-40", (1, 32, 40), (1, 8, 8), 2, 1, [(1, 4, 5)]),                          # 40, five each; at head dimension 128 four groups
    ("p96-45", (4, 18, 40), (2, 6, 8), 1, 2, [(1, 3, 5), (1, 1, 1)]),               # 45, five and six each; 3
    ("p32-49", (1, 28, 56), (1, 4, 8), 1, 2, [(1, 7, 7), (1, 1, 1)]),               # 49 and 1
    ("p160-45", (5, 24, 12), (5, 8, 4), 1, 1, [(1, 3, 3)]),
    ("p128-256-waves", (4, 32, 32), (2, 8, 8), 2, 1, [(2, 3, 3)]),                  # 72
    ("p384-108", (6, 24, 24), (6, 8, 8), 1, 2, [(1, 3, 3), (1, 1, 1)]),             # 108 and 12
]
SHORT = {("p64-40", 128)}
FOUR = [
    ("one wave more", (1, 64, 72), (1, 8, 8), 1, 2, [(1, 5, 5)]),                   # 288 waves
    ("36 sub-blocks", (4, 24, 24), (2, 8, 8), 1, 2, [(1, 3, 3)]),
    ("39 sub-blocks", (1, 12, 104), (1, 4, 8), 1, 2, [(1, 3, 13)]),
]


@pytest.mark.parametrize("D", [64, 128])
def test_eight_groups_for_long_walks_where_every_cu_has_at_most_one_workgroup(D):
    for name, grid, tile, B, H, windows in EIGHT:
        if (name, D) in SHORT:
            continue
        lines = launches(B, H, D, grid, tile, windows, gradients=True)
        assert [line.split(" items")[0] for line in lines] == ["dq_one_buffer<%d,1,8,1>" % D, "dkv<%d,1,8,1,1>" % D], (name, lines)
        # every workgroup has a CU of its own, and no order of the rows evens anything out
        assert lines[1].endswith(", head after head"), (name, lines)
    for name, grid, tile, B, H, windows in FOUR + [case for case in EIGHT if (case[0], D) in SHORT]:
        assert not any("<%d,1,8," % D in line for line in launches(B, H, D, grid, tile, windows, gradients=True)), name


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("name,grid,tile,B,H,windows", EIGHT, ids=[s[0] for s in EIGHT])
def test_gradients_of_eight_groups_match_the_oracle(name, grid, tile, B, H, windows, D):
    w = syn.custom("bwd-eight-" + name, B, H, D, grid, tile, [windows[h % len(windows)] for h in range(H)], "bf16", seed=1919)
    q, k, v = syn.make_qkv(w)
    g = syn.make_dout(w)
    (dq, dk, dv), _ = gpu_backward(w, q, k, v, g)
    for b, h in {(0, 0), (B - 1, H - 1)}:
        rq, rk, rv = oracle_backward(w, q, k, v, g, b, h)
        for label, got, ref in (("dQ", dq, rq), ("dK", dk, rk), ("dV", dv, rv)):
            assert_grad_parity(got[b, h].float().numpy(), ref, "%s D%d %s b%d h%d" % (name, D, label, b, h))
