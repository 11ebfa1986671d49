"""Finishing kernel of the mask search: partial sums of many slabs, and the choice among more patterns than a wave has lanes."""
import pytest
import torch

import paper_2502_04507_amd as sta

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GRID, TILE = (1, 16, 32), (1, 8, 8)


@pytest.mark.parametrize("B,H,n_patterns", [(1, 1, 1), (3, 5, 2), (19, 9, 64), (2, 70, 65), (1, 3, 200)])
def test_losses_and_first_minimum(B, H, n_patterns):
    g = torch.Generator(device=DEV).manual_seed(B * 100 + H)
    q, k, v = (torch.randn((B, H, 512, 64), generator=g, device=DEV).to(torch.bfloat16) for _ in range(3))
    kinds = [(1, 1, 1), (1, 1, 3), (1, 2, 1), (1, 1, 4)]
    patterns = [kinds[(i * 7 + i // 4) % 4] for i in range(n_patterns)]
    o_full, o_pattern = torch.empty_like(q), torch.empty_like(q)
    ws = torch.empty(sta.sta_head_mse_workspace_bytes(B, H), dtype=torch.uint8, device=DEV)
    losses = torch.full((n_patterns, H), float("nan"), device=DEV)
    best = torch.full((H,), -5, dtype=torch.int32, device=DEV)
    sta.sta_mask_search(q, k, v, GRID, TILE, patterns, o_full, o_pattern, ws, losses, best)
    # the last pattern's output is still there: its loss in 64 bits (the kernel sums 32-bit squares per lane: 2^-24 each)
    want = (o_full.double() - o_pattern.double()).square().mean(dim=(0, 2, 3))
    torch.testing.assert_close(losses[-1].double(), want, rtol=1e-5, atol=0)
    rows = losses.cpu()
    for i, p in enumerate(patterns):                                # the same pattern gives the same loss wherever it stands
        assert torch.equal(rows[i], rows[patterns.index(p)])
    for h in range(H):
        column = rows[:, h].tolist()
        assert best[h].item() == column.index(min(column))


def test_a_head_without_a_finite_loss_has_no_best_pattern():
    B, H = 2, 3
    q, k = (torch.randn((B, H, 512, 64), device=DEV).to(torch.bfloat16) for _ in range(2))
    v = torch.randn((B, H, 512, 64), device=DEV).to(torch.bfloat16)
    v[:, 1] *= 1e30                                                # finite (draws stay below 10), squared differences beyond fp32
    o_full, o_pattern = torch.empty_like(q), torch.empty_like(q)
    ws = torch.empty(sta.sta_head_mse_workspace_bytes(B, H), dtype=torch.uint8, device=DEV)
    losses, best = torch.zeros((2, H), device=DEV), torch.zeros((H,), dtype=torch.int32, device=DEV)
    sta.sta_mask_search(q, k, v, GRID, TILE, [(1, 1, 1), (1, 2, 1)], o_full, o_pattern, ws, losses, best)
    assert torch.isinf(losses[:, 1]).all() and torch.isfinite(losses[:, [0, 2]]).all()
    assert best.tolist()[1] == -1 and min(best.tolist()[0], best.tolist()[2]) >= 0
