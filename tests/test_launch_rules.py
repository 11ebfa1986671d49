"""Host-side rules of the forward and gradient launches: which item a workgroup id runs, where the last round of workgroups is
cut into parts.  No GPU: without one the rules count 256 compute units."""
import ctypes
import re

import numpy as np
import pytest

import paper_2502_04507_amd as sta
from tests import test_gpu_backward_eight_groups, test_gpu_backward_groups, test_gpu_backward_launches, test_gpu_backward_single_waves
from tests import test_gpu_forward_groups, test_gpu_forward_large
from tests import test_gpu_forward_launches
from tests.launch_shapes import launches

CUS = 256


@pytest.mark.parametrize("per_head", [1, 2, 3, 7, 8, 9, 25, 36, 41, 108, 300, 1201])
def test_every_workgroup_id_names_an_item_and_the_xcds_get_equal_shares(per_head):
    for slices in (1, 2, 3, 7, 8, 9, 24, 48, 333):
        total = per_head * slices
        items = np.full(total + 1, 0xffffffff, dtype=np.uint32)
        sta.load_library().sta_dealt_items(per_head, slices, ctypes.c_void_p(items.ctypes.data))
        assert items[total] == 0xffffffff
        items = items[:total]
        assert np.array_equal(np.sort(items), np.arange(total)), (per_head, slices)
        # ids go to the XCDs in turn, so their shares are equal as they are; each takes runs of about an eighth of a head
        share = items[::8]
        runs = 1 + np.count_nonzero(np.diff(share.astype(np.int64)) != 1)
        assert runs <= -(-total // (8 * -(-per_head // 8))) + 1, (per_head, slices, runs)


@pytest.mark.parametrize("grid,window", [((12, 24, 40), (1, 3, 3)), ((6, 48, 80), (1, 3, 3)), ((18, 48, 48), (3, 3, 3)),
                                         ((6, 40, 40), (1, 3, 3)), ((30, 48, 80), (3, 3, 3)), ((18, 24, 24), (1, 1, 1))])
def test_a_last_round_of_at_most_half_is_cut_into_parts(grid, window):
    """384-token tiles, head dimension 128, with a workspace: one workgroup of 12 waves per tile and CU."""
    per_head = grid[0] * grid[1] * grid[2] // 384
    cut = 0
    for heads in range(1, 97):
        items = per_head * heads
        tail = items % CUS
        if items < CUS or tail == 0 or 2 * tail > CUS:
            continue
        (line,) = launches(1, heads, 128, grid, (6, 8, 8), [window], workspace=True)
        match = re.fullmatch(r"x32<12> items %d workgroups (\d+) parts (\d+) of (\d+)" % items, line)
        assert match, line
        workgroups, parts, of = map(int, match.groups())
        units = 12 * np.prod([min(2 * (w // 2) + 1, g // t) for w, g, t in zip(window, grid, (6, 8, 8))])
        want = min(CUS // tail, max(p for p in range(1, units + 1) if units // p >= 4))
        assert (parts, of, workgroups) == (want, tail, items - tail + tail * want), line
        cut += 1
    assert cut > 10


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("grid,heads,windows", [
    ((6, 24, 24), 10, [(1, 2, 3), (1, 3, 2), (1, 1, 2), (1, 2, 3), (1, 3, 3)]),      # 24 rows of long walks, six of short ones
    ((6, 8, 48), 9, [(1, 1, 5)]),                                                    # nine rows
    ((6, 24, 24), 14, [(1, 3, 3)]), ((12, 24, 40), 3, [(1, 3, 3), (2, 1, 1)]),
])
def test_the_xcds_of_a_gradient_launch_walk_equally_far(grid, heads, windows, D):
    """Counted in sub-blocks of 32 tokens, over the walks that the windows give their heads."""
    for line in launches(1, heads, D, grid, (6, 8, 8), windows, gradients=True):
        most, total = map(int, re.search(r"fullest XCD (\d+) of (\d+)", line).groups())
        assert most <= 1.06 * total / 8, line         # chunks may leave a twentieth


@pytest.mark.parametrize("B,H,grid,windows,want", [
    (7, 20, (1, 16, 24), [(1, 2, 1), (1, 2, 3), (1, 2, 3)], "dkv_pair<2,1,1>"),       # 1680 waves, by their walks 1288
    (4, 20, (1, 16, 48), [(1, 2, 1), (1, 1, 2)], "dkv_pair<2,1,1>"),                  # 1920, 1600
    (7, 8, (1, 48, 32), [(1, 3, 1), (1, 1, 1), (1, 1, 1), (1, 5, 3)], "dkv<128,2,2,1,1>"),     # 2688, 896; one long walk
    (1, 25, (1, 32, 48), [(1, 3, 1), (1, 4, 2), (1, 3, 2)], "dkv<128,2,2,1,1>"),      # 1200, 780; walks of up to 32 of 12 on average
    (1, 25, (1, 32, 48), [(1, 3, 1)], "dkv_pair<2,1,1>"),                             # 1200, equal
    (4, 25, (1, 32, 48), [(1, 3, 1)], "dkv<128,2,1,1,1>"),                            # 4800
])
def test_short_walks_on_64_token_tiles_count_by_their_length(B, H, grid, windows, want):
    assert launches(B, H, 128, grid, (1, 8, 8), windows, gradients=True)[1].startswith(want + " ")


@pytest.mark.parametrize("H,grid,window,want", [
    (31, (6, 16, 16), (1, 2, 2), "dkv_pair<6,1,1>"), (14, (6, 24, 24), (1, 3, 3), "dkv_pair<6,1,1>"),      # one round, equal walks
    (2, (30, 24, 32), (3, 3, 3), "dkv<128,2,2,1,1>"), (7, (6, 32, 32), (1, 3, 3), "dkv<128,2,2,1,1>"),     # key tiles of 2.2 and 1.8 times the walk
    (16, (6, 24, 24), (1, 3, 3), "dkv<128,4,1,1,1>"), (3, (18, 24, 48), (3, 3, 3), "dkv<128,4,1,1,1>"),    # beyond a round of pairs
    (4, (12, 32, 40), (1, 3, 3), "dkv<128,2,2,1,1>"), (7, (6, 48, 40), (1, 3, 3), "dkv<128,2,2,1,1>"),     # one walk of 2.4 and 1.8 shares
])
def test_launches_of_a_round_or_so_go_by_the_longest_walk_of_a_key_tile(H, grid, window, want):
    assert launches(1, H, 128, grid, (6, 8, 8), [window], gradients=True)[1].startswith(want + " ")


@pytest.mark.parametrize("D,H,grid,tile,windows,want", [
    (64, 9, (1, 96, 96), (1, 8, 8), [(1, 12, 12), (1, 3, 3), (1, 1, 3)], "dq<64,2,2,1> dkv<64,2,2,1,1>"),      # longest 3.4 times a place's share
    (128, 9, (1, 96, 96), (1, 8, 8), [(1, 12, 12), (1, 3, 3), (1, 1, 3)], "dq<128,2,2,1> dkv<128,2,2,1,1>"),   # 2.2
    (64, 4, (12, 48, 48), (6, 8, 8), [(1, 1, 3), (1, 3, 3), (1, 1, 1), (2, 6, 6)], "dq<64,2,2,1> dkv<64,2,2,1,1>"),    # 3.0; by walks 1020 waves
    (64, 8, (12, 48, 48), (6, 8, 8), [(1, 1, 3), (1, 3, 3), (1, 1, 1), (2, 6, 6)], "dq<64,4,1,1> dkv<64,4,1,2,1>"),    # 1.5; 2040
    (128, 6, (9, 40, 40), (3, 8, 8), [(3, 3, 3), (1, 1, 3), (1, 1, 1)], "dq<128,3,1,1> dkv<128,2,2,1,1>"),     # 1.5 of six waves a CU
    (128, 2, (9, 40, 40), (3, 8, 8), [(3, 3, 3), (1, 5, 5)], "dq<128,3,1,1> dkv<128,2,2,1,1>"),                # 900 waves; 1.77 of six a CU
    (128, 6, (18, 12, 32), (6, 6, 8), [(3, 2, 3), (3, 1, 1)], "dq<128,3,1,1> dkv<128,1,4,1,1>"),               # 2.03, the long ones 0.42 of the places
    (128, 4, (3, 48, 40), (3, 8, 8), [(1, 6, 5), (1, 3, 5), (1, 6, 5), (1, 3, 3)], "dq<128,3,2,1> dkv<128,1,4,1,1>"),  # 720; 2.1 and more
    (64, 14, (3, 48, 40), (3, 8, 8), [(1, 6, 5)] * 4 + [(1, 5, 5)] * 3 + [(1, 3, 5)] * 3 + [(1, 1, 3)] * 4, "dq<64,3,1,1> dkv<64,2,2,1,1>"),  # 2.03, 0.41
    (64, 6, (3, 48, 80), (3, 8, 8), [(1, 6, 10), (1, 1, 3), (1, 1, 3)], "dq<64,3,2,1> dkv<64,2,2,1,1>"),       # 3.6
    (128, 12, (6, 16, 72), (6, 8, 8), [(1, 2, 5), (1, 1, 3), (1, 2, 1), (1, 2, 1)], "dq<128,4,1,1> dkv<128,4,1,1,1>"),  # 1.86 of eight a CU
    (64, 4, (16, 32, 40), (4, 8, 8), [(4, 4, 5), (1, 3, 3)], "dq<64,2,2,1> dkv<64,2,2,1,1>"),
    (64, 160, (4, 72, 8), (2, 8, 8), [(2, 9, 1), (2, 3, 1), (2, 3, 1), (2, 1, 1)], "dq<64,4,1,1> dkv<64,4,1,2,1>"),    # 11520 waves, by walks 5120
    (64, 80, (4, 72, 8), (2, 8, 8), [(2, 9, 1), (2, 3, 1), (2, 3, 1), (2, 1, 1)], "dq<64,4,1,1> dkv<64,2,2,1,1>"),     # 5760
    (64, 6, (12, 32, 32), (6, 8, 8), [(2, 4, 4), (1, 3, 3), (1, 1, 3)], "dq<64,2,2,1> dkv<64,2,2,1,1>"),       # 2304, by walks 1056
    (64, 16, (1, 64, 64), (1, 8, 8), [(1, 5, 5)], "dq<64,2,2,1> dkv<64,1,4,1,1>"),                             # 2048 equal walks of 50
    (64, 16, (1, 64, 64), (1, 8, 8), [(1, 3, 3)], "dq<64,2,1,1> dkv<64,2,2,1,1>"),                             # of 18
])
def test_long_walks_among_short_ones_are_halved_in_the_gradients(D, H, grid, tile, windows, want):
    assert kernels(launches(1, H, D, grid, tile, windows, gradients=True)) == want.split(" ")


@pytest.mark.parametrize("H,grid,tile,windows,want", [
    (1, (18, 24, 24), (6, 8, 8), [(1, 3, 3)], "solo<64,3,12,0> items 216"),
    (6, (18, 8, 16), (6, 8, 8), [(3, 1, 2)] * 3 + [(3, 1, 1)] + [(1, 1, 2)] * 2, "solo<64,4,8,0> items 216"),      # 432, by their walks 360
    (2, (3, 40, 48), (3, 8, 8), [(1, 5, 5), (1, 3, 3)], "solo<64,3,12,0> items 240"),              # 360 waves of 150 and 54 units
    (3, (12, 16, 32), (6, 8, 8), [(2, 2, 4), (2, 2, 3), (1, 1, 3)], "solo<64,4,8,0> items 288"),   # 576, by their walks 384
    (25, (3, 40, 48), (3, 8, 8), [(1, 5, 6)] + [(1, 1, 1)] * 24, "solo<64,4,8,0> items 2250"),     # 4500, by their walks 360
])
def test_twelve_waves_for_48_queries_where_no_cu_gets_two_workgroups(H, grid, tile, windows, want):
    assert launches(1, H, 64, grid, tile, windows) == [want]


@pytest.mark.parametrize("B,H,grid,windows,want", [
    (1, 2, (12, 48, 48), [(1, 3, 3)], "x32<4> items 432"),            # workgroups of twelve waves fill 0.56 of a round
    (1, 3, (12, 24, 88), [(1, 3, 3)], "x32<12> items 198"),           # 0.77
    (1, 4, (30, 8, 80), [(5, 1, 7)], "x32<12> items 200"),            # 0.78, long walks
    (1, 3, (12, 48, 48), [(1, 3, 3)], "x32<12> items 216"),           # 0.84
    (1, 4, (12, 48, 48), [(1, 3, 3)], "x32<4> items 864"),            # 1.13 rounds
    (1, 8, (12, 32, 48), [(1, 3, 3)], "x32<4> items 1152"),           # 1.5
    (1, 6, (12, 48, 48), [(1, 3, 3)], "x32<12> items 432"),           # 1.69
    (1, 8, (12, 48, 48), [(1, 3, 3)], "x32<4> items 1728"),           # 2.25
    (1, 12, (12, 48, 48), [(1, 3, 3)], "x32<12> items 864"),          # 3.38
    (1, 12, (6, 40, 48), [(1, 3, 1), (1, 3, 5)], "x32<12> items 360"),        # 1.41 and half of it 36 units of 180: long ones 0.70 of a round
    (1, 20, (6, 40, 32), [(1, 5, 4), (1, 1, 3)], "x32<12> items 400"),        # 1.56, 36 of 240: 0.78
    (2, 8, (12, 96, 8), [(2, 11, 1), (2, 3, 1)], "x32<12> items 384"),        # 1.5, 72 of 264: 0.75; longest 1.048 shares
    (1, 7, (6, 56, 48), [(1, 3, 1), (1, 3, 1), (1, 1, 1)], "x32<4> items 882"),       # 1.15, 12 of 36: 0.82
    (1, 12, (6, 40, 48), [(1, 3, 1), (1, 3, 5), (1, 3, 3)], "x32<4> items 1080"),     # 1.41, 36, 180 and 108: 0.47
    (1, 12, (6, 40, 48), [(1, 3, 3), (1, 3, 5)], "x32<4> items 1080"),        # 1.41, 108 of 180: 1.1 rounds of work
    (1, 16, (6, 32, 72), [(1, 1, 5), (1, 3, 9), (1, 3, 1)], "x32<4> items 1728"),     # 2.25, 60, 324 and 36
])
def test_twelve_waves_a_workgroup_where_their_rounds_are_full_enough(B, H, grid, windows, want):
    """384-token tiles, head dimension 128, no workspace."""
    (line,) = launches(B, H, 128, grid, (6, 8, 8), windows)
    assert line.startswith(want + " "), line


@pytest.mark.parametrize("H,grid,windows,workspace,want", [
    (4, (12, 48, 48), [(1, 1, 3), (1, 3, 3), (1, 1, 1), (2, 6, 6)], False, "x32<4> items 864 workgroups 864 parts 1"),     # longest 3.0 shares
    (8, (12, 48, 48), [(1, 1, 3), (1, 3, 3), (1, 1, 1), (2, 6, 6)], False, "x32<4> items 1728 workgroups 1728 parts 1"),   # 1.5
    (12, (12, 48, 48), [(1, 1, 3), (1, 3, 3), (1, 1, 1), (2, 6, 6)], False, "x32<12> items 864 workgroups 864 parts 1"),   # 1.0
    (3, (18, 40, 40), [(3, 3, 3), (3, 3, 3), (3, 3, 5)], False, "x32<4> items 675 workgroups 675 parts 1"),    # 0.88 rounds, 324 and 540 units
    (5, (36, 48, 8), [(6, 3, 1), (5, 3, 1)], False, "x32<12> items 180 workgroups 180 parts 1"),               # 0.70, 216 and 180
    (8, (24, 32, 8), [(4, 4, 1), (4, 4, 1), (2, 4, 1)], True, "x32<12> items 128 workgroups 256 parts 2"),     # 0.5, 192 and 144
    (12, (12, 32, 32), [(1, 3, 3), (2, 4, 4), (1, 1, 3)], True, "x32<4> items 1152 workgroups 1152 parts 1"),  # 108, 384 and 36
    (12, (12, 32, 32), [(1, 3, 3)], True, "x32<12> items 384 workgroups 512 parts 2"),                         # equal
])
def test_four_waves_a_workgroup_where_the_launch_waits_for_long_walks(H, grid, windows, workspace, want):
    """384-token tiles, head dimension 128."""
    (line,) = launches(1, H, 128, grid, (6, 8, 8), windows, workspace=workspace)
    assert line.startswith(want + " of "), line


@pytest.mark.parametrize("H,grid,tile,windows,want", [
    (32, (1, 64, 64), (1, 8, 8), [(1, 3, 3)], "group<128,2,1,1,1> items 2048"),         # 2.0 rounds of four two-wave workgroups a CU
    (24, (1, 64, 64), (1, 8, 8), [(1, 3, 3)], "group_one_v<128,2,1,1,1> items 1536"),   # 1.5
    (25, (1, 64, 64), (1, 8, 8), [(1, 3, 3)], "group<128,2,1,1,1> items 1600"),         # 1.56
    (16, (1, 80, 80), (1, 8, 8), [(1, 5, 5)], "group<128,2,1,1,1> items 1600"),
    (20, (1, 64, 64), (1, 8, 8), [(1, 3, 3)], "group_one_v<128,2,1,1,1> items 1280"),   # 1.25
    (16, (1, 64, 64), (1, 8, 8), [(1, 3, 3)], "group<128,2,1,1,1> items 1024"),         # 1.0
    (10, (1, 64, 64), (1, 8, 8), [(1, 3, 3)], "group_one_v<128,2,2,1,1> items 640"),
    (8, (1, 64, 64), (1, 8, 8), [(1, 3, 3)], "group<128,2,2,1,1> items 512"),
    (40, (1, 64, 64), (1, 8, 8), [(1, 3, 3)], "group_one_v<128,2,1,1,1> items 2560"),   # 2.5
    (18, (1, 96, 96), (1, 8, 8), [(1, 3, 3), (1, 5, 5), (1, 12, 12)], "group<128,2,2,1,1> items 2592"),       # by walks 1.2 rounds
    (9, (1, 96, 96), (1, 8, 8), [(1, 3, 3), (1, 5, 5), (1, 12, 12)], "group_one_v<128,2,2,1,1> items 1296"),  # 0.6
    # heads of different walks: rounds of those over half the longest, and the longest in even shares of a place
    (36, (1, 64, 64), (1, 8, 8), [(1, 3, 3), (1, 1, 1), (1, 1, 1)], "group<128,2,1,1,1> items 2304"),         # 0.75, 1.1
    (48, (1, 64, 64), (1, 8, 8), [(1, 3, 3), (1, 1, 1), (1, 1, 1)], "group_one_v<128,2,1,1,1> items 3072"),   # 1.0, 0.8
    (40, (1, 64, 64), (1, 8, 8), [(1, 3, 3), (1, 1, 1)], "group_one_v<128,2,1,1,1> items 2560"),              # 1.25
    (84, (1, 48, 40), (1, 8, 8), [(1, 6, 5), (1, 2, 5), (1, 1, 3), (1, 1, 3)], "group<128,2,1,1,1> items 2520"),      # 0.6, 0.96
    (60, (1, 64, 64), (1, 8, 8), [(1, 3, 3), (1, 1, 1)], "group<128,2,1,1,1> items 3840"),                    # 1.9, 0.48
    (64, (1, 64, 64), (1, 8, 8), [(1, 3, 3), (1, 1, 3)], "group_one_v<128,2,1,1,1> items 4096"),              # 2.0, 0.37
    (70, (1, 64, 64), (1, 8, 8), [(1, 3, 3), (1, 1, 1)], "group_one_v<128,2,1,1,1> items 4480"),              # 2.2
    (40, (1, 64, 64), (1, 8, 8), [(1, 3, 3), (1, 2, 3)], "group_one_v<128,2,1,1,1> items 2560"),              # all of them, 2.5
    (10, (20, 16, 16), (5, 8, 8), [(3, 2, 2)] * 7 + [(4, 2, 1)] * 3, "group<128,2,1,1,1> items 800"),         # two groups: by walks 720, long 800
    # tiles of 32 tokens
    (80, (1, 16, 16), (1, 4, 8), [(1, 3, 1)], "group<128,1,1,1,1> items 640"),
    (140, (1, 16, 16), (1, 4, 8), [(1, 3, 1)], "group_one_v<128,1,1,1,1> items 1120"),                        # 1.1
    (140, (1, 16, 16), (1, 4, 8), [(1, 3, 1), (1, 1, 1)], "group<128,1,1,1,1> items 1120"),                   # 0.55, 1.4
    (220, (1, 16, 16), (1, 4, 8), [(1, 3, 1)], "group<128,1,1,1,1> items 1760"),                              # 1.7
    (220, (1, 16, 16), (1, 4, 8), [(1, 3, 2), (1, 1, 1), (1, 3, 2)], "group<128,1,1,1,1> items 1760"),        # 1.15, but 1.7 in all
    (170, (1, 16, 16), (1, 4, 8), [(1, 3, 2), (1, 1, 1), (1, 3, 2), (1, 3, 2), (1, 3, 2)], "group_one_v<128,1,1,1,1> items 1360"),   # 1.06
])
def test_one_lds_stage_of_v_by_the_rounds_of_the_launch(H, grid, tile, windows, want):
    assert launches(1, H, 128, grid, tile, windows) == [want]


@pytest.mark.parametrize("H,grid,tile,windows,want", [                                  # waves, units
    (1, (12, 24, 24), (6, 8, 8), [(2, 3, 3)], "solo<128,2,8,0> items 216"),             # 216, 216
    (2, (12, 24, 24), (6, 8, 8), [(2, 3, 3)], "group<128,2,4,0,1> items 216"),          # 432, 216
    (1, (18, 24, 24), (6, 8, 8), [(3, 3, 3)], "x32<12> items 27 "),                     # 324, 324
    (1, (12, 48, 48), (6, 8, 8), [(1, 3, 3)], "group<128,2,2,0,1> items 432"),          # 864, 108
    (3, (12, 24, 32), (6, 8, 8), [(2, 2, 4)], "x32<12> items 72 "),                     # 864, 288
    (5, (12, 24, 24), (6, 8, 8), [(1, 3, 3)], "x32<12> items 90 "),                     # 1080, 108
    (2, (2, 72, 48), (2, 8, 8), [(1, 9, 6)], "group<128,2,4,0,1> items 216"),           # 432, 216
    (1, (24, 24, 16), (6, 8, 8), [(3, 3, 2)], "x32<12> items 24 "),                     # 288, 216
    (1, (24, 24, 16), (6, 8, 8), [(4, 3, 1)], "group<128,2,4,0,1> items 144"),          # 288, 144
    (2, (12, 88, 8), (6, 8, 8), [(2, 5, 1)], "x32<12> items 44 "),                      # 528, 120
    (3, (6, 80, 16), (6, 8, 8), [(1, 5, 2)], "group<128,2,2,0,1> items 360"),           # 720, 120
    (2, (12, 24, 48), (6, 8, 8), [(1, 3, 3)], "group<128,2,2,0,1> items 432"),          # 864, 108
    (2, (2, 72, 48), (2, 8, 8), [(1, 9, 6), (1, 1, 6)], "x32<4> items 108 "),           # 432, 216 and 24
    (2, (20, 8, 40), (4, 8, 8), [(5, 1, 5), (5, 1, 1)], "x32<4> items 100 "),           # 400, 200 and 40
    (2, (4, 48, 40), (2, 8, 8), [(2, 6, 5), (2, 5, 5)], "group<128,2,4,0,1> items 240"),    # 480, 240 and 200
    (2, (4, 72, 24), (4, 8, 8), [(1, 5, 3), (1, 1, 3)], "group<128,2,4,0,1> items 216"),    # 432, 120 and 24
])
def test_key_groups_where_a_workspace_is_given(H, grid, tile, windows, want):
    (line,) = launches(1, H, 128, grid, tile, windows, workspace=True)
    assert line.startswith(want), line


# The kernels that the cases of tests/test_gpu_forward_launches.py and test_gpu_backward_launches.py run: a rule that sends one of
# them elsewhere leaves its kernel without those tests.
FORWARD = {
    "own-p64-32q-8": "solo<64,2,8,0>", "own-p64-32q-4": "solo<64,2,4,0>", "own-p64-64q-8": "solo<64,4,8,0>",
    "own-p64-64q-4": "solo<64,4,4,0>", "own-p192-64q-4": "solo<64,4,4,0>", "own-p384-64q-8": "solo<64,4,8,0>",
    "own-p96-4": "solo<64,2,4,1>", "own-p32-4": "solo<64,2,4,1>", "own-p160-8": "solo<64,2,4,1>",
    "own-p384-d128-8": "solo<128,2,8,0>", "own-p128-d128-4": "solo<128,2,4,0>", "own-p64-d128-4": "solo<128,2,4,1>",
    "own-p192-d128-4": "solo<128,2,4,1>", "own-p32-d128-4": "solo<128,2,4,1>",
    "shared-p64-two": "group<64,2,2,0,1>", "shared-p64-one": "group<64,2,1,0,1>", "shared-p192-two": "group<64,2,2,0,1>",
    "shared-p192-three-two": "group<64,3,2,0,1>", "shared-p192-three-one": "group<64,3,1,0,1>", "shared-p96": "group<64,3,1,1,1>",
    "shared-p32-two": "group<64,1,2,1,1>", "shared-p32-one": "group<64,1,1,1,1>", "shared-p384-d128-four": "group<128,2,4,0,1>",
    "shared-p384-d128-two": "group<128,2,2,0,1>", "shared-p384-d128-one": "group<128,2,1,0,1>",
    "shared-p64-d128-two": "group<128,2,2,1,1>", "shared-p64-d128-one": "group<128,2,1,1,1>",
    "shared-p96-d128-two": "group<128,3,2,1,1>", "shared-p96-d128-one": "group<128,3,1,1,1>", "shared-p32-d128": "group<128,1,1,1,1>",
    "own-p384-48q-12": "solo<64,3,12,0>", "own-p192-48q-12": "solo<64,3,12,0>",
    "one-v-p64-d128-two": "group_one_v<128,2,2,1,1>", "one-v-p64-d128-one": "group_one_v<128,2,1,1,1>",
    "one-v-p320-d128": "group_one_v<128,2,1,1,1>", "one-v-p64-d128-short": "group_one_v<128,2,1,1,1>",
    "one-v-p32-d128": "group_one_v<128,1,1,1,1>", "one-v-p32-d128-short": "group_one_v<128,1,1,1,1>",
}
BACKWARD = {
    ("p128-two-groups", 64): "dq<64,2,2,1> dkv<64,2,2,1,1>", ("p128-two-groups", 128): "dq<128,2,2,1> dkv<128,2,2,1,1>",
    ("p384-four-waves", 64): "dq<64,4,1,1> dkv<64,4,1,2,1>", ("p384-four-waves", 128): "dq<128,4,1,1> dkv<128,4,1,1,1>",
    ("p128-four-waves", 64): "dq<64,4,1,1> dkv<64,4,1,2,1>", ("p128-four-waves", 128): "dq<128,4,1,1> dkv<128,4,1,1,1>",
    ("p64-two-groups", 64): "dq<64,2,1,1> dkv<64,2,2,1,1>", ("p64-two-groups", 128): "dq<128,2,1,1> dkv<128,2,2,1,1>",
    ("p64-two-pairs", 128): "dq<128,2,1,1> dkv_pair<2,1,1>", ("p384-mixed", 128): "dq<128,4,1,1> dkv<128,2,2,1,1>",
    ("p384-six-pairs", 128): "dq<128,4,1,1> dkv_pair<6,1,1>", ("p64-two-waves", 64): "dq<64,2,1,1> dkv<64,2,1,1,1>",
    ("p64-two-waves", 128): "dq<128,2,1,1> dkv<128,2,1,1,1>", ("p192-two-groups", 64): "dq<64,3,1,1> dkv<64,2,2,1,1>",
    ("p192-two-groups", 128): "dq<128,3,1,1> dkv<128,2,2,1,1>", ("p96-many", 64): "dq<64,3,1,1> dkv<64,3,1,1,1>",
    ("p96-many", 128): "dq<128,3,1,1> dkv_pair<3,2,1>", ("p96-some", 64): "dq<64,3,1,1> dkv<64,1,4,1,1>",
    ("p96-some", 128): "dq<128,3,1,1> dkv_pair<3,2,1>", ("p96-few", 128): "dq_one_buffer<128,1,4,1> dkv<128,1,4,1,1>",
    ("p192-three-two", 128): "dq<128,3,2,1> dkv<128,2,2,1,1>",
    ("p32-some", 64): "dq<64,1,1,1> dkv<64,1,2,1,1>", ("p32-some", 128): "dq<128,1,1,1> dkv_pair<1,1,1>",
    ("p32-many", 64): "dq<64,1,1,1> dkv<64,1,1,1,1>", ("p32-many", 128): "dq_one_buffer<128,1,1,1> dkv_pair<1,1,1>",
}
# ... and the shapes that other GPU tests run: test_gpu_forward_groups.py (two units per stage), test_gpu_forward_large.py,
# test_gpu_backward_groups.py (three waves in two groups), test_gpu_backward_eight_groups.py, test_gpu_backward_single_waves.py
ELSEWHERE = {"group<64,4,1,0,2>", "x32<4>", "x32<12>", "solo<64,2,8,1>", "solo<128,2,8,1>", "dq<64,3,2,1>", "dq<64,1,4,1>", "dq<128,1,4,1>",
             "dq_one_buffer<64,1,4,1>", "dq_one_buffer<64,1,8,1>", "dq_one_buffer<128,1,8,1>", "dkv<64,1,8,1,1>", "dkv<128,1,8,1,1>", "dq_one_buffer<64,1,1,1>"}


def kernels(lines):
    return [line.split(" ")[0] for line in lines]


def test_the_gpu_tests_run_the_kernels_that_they_are_for():
    for name, D, grid, tile, heads, window in test_gpu_forward_launches.LAUNCHES:
        assert kernels(launches(1, heads, D, grid, tile, [window])) == [FORWARD[name]], name
    for name, D, grid, tile, B, H, windows in test_gpu_backward_launches.CASES:
        assert kernels(launches(B, H, D, grid, tile, windows, gradients=True)) == BACKWARD[name, D].split(" "), (name, D)
    seen = set()
    for _, grid, tile, windows in test_gpu_forward_groups.SHAPES:
        for D in (64, 128):
            seen.update(kernels(launches(1, len(windows), D, grid, tile, windows)))
    for heads, grid, tile in ((30, (6, 16, 24), (6, 8, 8)), (66, (4, 16, 16), (2, 8, 8))):
        seen.update(kernels(launches(1, heads, 64, grid, tile, [(1, 3, 3), (3, 3, 3)])))
    for name, (grid, tile, heads, workspace) in test_gpu_forward_large.LAUNCHES.items():
        (line,) = launches(1, heads, 128, grid, tile, [(1, 3, 3), (3, 3, 3)], workspace=workspace)
        assert ("parts 1 " not in line) == workspace, (name, line)
        seen.update(kernels([line]))
    for _, grid, tile, B, H, windows in test_gpu_backward_groups.SHAPES:
        for D in (64, 128):
            seen.update(kernels(launches(B, H, D, grid, tile, windows, gradients=True)))
    single = test_gpu_backward_single_waves
    for D, grid, tile, B, H, windows in ([(D, *rest) for _, *rest in test_gpu_backward_eight_groups.EIGHT for D in (64, 128)]
                                         + [(D, *rest) for _, dims, *rest in single.SINGLE for D in dims]
                                         + [(D, grid, tile, 1, H, windows) for _, D, grid, tile, H, windows in single.KEYS]
                                         + [case[1:] for case in single.ALONE]):
        seen.update(kernels(launches(B, H, D, grid, tile, windows, gradients=True)))
    assert ELSEWHERE <= seen, ELSEWHERE - seen
    assert {"dkv_pair<6,1,1>", "dkv<128,4,1,1,1>", "dkv<128,2,2,1,1>"} == {
        kernels(launches(1, H, 128, grid, (6, 8, 8), windows, gradients=True))[1] for _, grid, H, windows in test_gpu_backward_groups.SIX_PAIRS}


def test_no_shape_is_without_a_gpu_test():
    """Launches drawn over the whole range take no shape that the tables above do not name."""
    named = set(FORWARD.values()) | {k for v in BACKWARD.values() for k in v.split(" ")} | ELSEWHERE
    rng = np.random.default_rng(7)
    tiles = [(6, 8, 8), (1, 8, 8), (2, 8, 8), (3, 8, 8), (4, 8, 8), (2, 6, 8), (4, 4, 6), (4, 4, 8), (5, 8, 8), (1, 4, 8), (6, 8, 16), (7, 4, 8)]
    seen = set()
    for _ in range(3000):
        tile = tiles[rng.integers(len(tiles))]
        n = [int(rng.integers(1, 4)) if tile[0] > 1 else 1, int(rng.integers(1, 7)), int(rng.integers(1, 9))]
        windows = [tuple(int(rng.integers(1, m + 1)) for m in n) for _ in range(rng.integers(1, 4))]
        B, H, D = int(rng.integers(1, 5)), int(np.exp(rng.uniform(0, 4))), int(rng.choice([64, 128]))
        args = (B, H, D, tuple(a * b for a, b in zip(n, tile)), tile, windows)
        seen.update(kernels(launches(*args, workspace=bool(rng.integers(2)))) + kernels(launches(*args, gradients=True)))
    assert seen <= named, seen - named
    assert named <= seen, named - seen
