"""Host-side rules of the forward and gradient launches: which item a workgroup id runs, where the last round of workgroups is
cut into parts.  No GPU: without one the rules count 256 compute units."""
import ctypes
import re

import numpy as np
import pytest

import paper_2502_04507_amd as sta
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
