"""GPU parity of the dK/dV kernel shapes that launches take once the smallest shapes (a wave per walk group) no longer serve them;
counts of waves are on 256 CUs.  Every slice runs, the oracle looks at three of them.  (test_launch_rules.py says which kernels each
of them runs.)"""
import pytest

import synth_inputs as syn
from tests.test_gpu_backward import assert_grad_parity, gpu_backward, oracle_backward

pytestmark = pytest.mark.gpu

LAUNCHES = [
    # name, head dimensions, grid, tile, batch, heads, windows
    ("p128-two-groups", (64, 128), (4, 16, 24), (2, 8, 8), 2, 8, [(2, 1, 3), (1, 1, 1)]),         # 768 waves
    ("p384-four-waves", (64, 128), (6, 16, 16), (6, 8, 8), 1, 36, [(1, 2, 1), (1, 1, 1)]),        # 1728
    ("p128-four-waves", (64, 128), (2, 8, 24), (2, 8, 8), 4, 132, [(1, 1, 3), (1, 1, 1)]),        # 6336
    ("p64-two-groups", (64, 128), (1, 16, 24), (1, 8, 8), 8, 8, [(1, 2, 3), (1, 1, 1)]),          # 768; 12 and 2 sub-blocks
    ("p64-two-pairs", (128,), (1, 16, 24), (1, 8, 8), 10, 10, [(1, 2, 3), (1, 1, 1)]),            # 1200; 12 and 2 sub-blocks
    ("p384-mixed", (128,), (6, 16, 16), (6, 8, 8), 1, 28, [(1, 2, 1), (1, 1, 1)]),                # 1344: no six pairs
    ("p384-six-pairs", (128,), (6, 16, 16), (6, 8, 8), 1, 28, [(1, 2, 1)]),                       # 1344
    ("p64-two-waves", (64, 128), (1, 16, 24), (1, 8, 8), 12, 15, [(1, 2, 2)]),                    # 2160
    ("p192-two-groups", (64, 128), (3, 16, 24), (3, 8, 8), 8, 9, [(1, 3, 2)]),                    # 2592; 36 sub-blocks
    ("p96-many", (64, 128), (2, 12, 16), (2, 6, 8), 4, 100, [(1, 1, 2), (1, 2, 1)]),              # 4800
    ("p96-some", (64, 128), (2, 12, 16), (2, 6, 8), 4, 33, [(1, 2, 2), (1, 1, 1)]),               # 1584
    ("p96-few", (128,), (4, 18, 40), (2, 6, 8), 1, 4, [(1, 3, 3), (1, 1, 1)]),                    # 360; 27 sub-blocks and 3
    ("p192-three-two", (128,), (3, 16, 40), (3, 8, 8), 1, 12, [(1, 1, 5), (1, 1, 1)]),            # 720; 30 and 6
    ("p32-some", (64, 128), (1, 8, 24), (1, 4, 8), 10, 10, [(1, 2, 3), (1, 1, 1)]),               # 600; 6 sub-blocks and 1
    ("p32-many", (64, 128), (1, 8, 24), (1, 4, 8), 20, 10, [(1, 1, 3)]),                          # 1200
]
CASES = [(name, D, *rest) for name, Ds, *rest in LAUNCHES for D in Ds]


@pytest.mark.parametrize("name,D,grid,tile,B,H,windows", CASES, ids=["%s-d%d" % c[:2] for c in CASES])
def test_launches_match_the_oracle(name, D, grid, tile, B, H, windows):
    w = syn.custom("bwd-launch-" + name, B, H, D, grid, tile, [windows[h % len(windows)] for h in range(H)], "bf16", seed=1717)
    q, k, v = syn.make_qkv(w)
    g = syn.make_dout(w)
    (dq, dk, dv), _ = gpu_backward(w, q, k, v, g)
    for b, h in ((0, 0), (B // 2, 1), (B - 1, H - 1)):
        rq, rk, rv = oracle_backward(w, q, k, v, g, b, h)
        for label, got, ref in (("dQ", dq, rq), ("dK", dk, rk), ("dV", dv, rv)):
            assert_grad_parity(got[b, h].float().numpy(), ref, "%s D%d %s b%d h%d" % (name, D, label, b, h))
