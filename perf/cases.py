"""What users of this package have it do, as cases that can be timed and compared: attention layers as they run at
inference, training steps through them, and the mask search that chooses windows.  Everything goes through the public
entry points of paper_2502_04507_amd, on tensors resident in GPU memory.

A case is a dict of plain values:
  kind     "layer":  tile_permute(Q, K, V) -> forward (with its workspace) -> untile(O), one attention layer;
           "train":  the same with forward_lse, then tile_permute(dO) -> backward -> untile(dQ, dK, dV);
           "search": mask_search on tensors already in tiled order (the full pass, one pass per pattern, the losses).
  B, H, D  batch, heads, head dimension
  grid, tile  "TxHxW" in tokens
  windows  "TxHxW" in tiles, a comma-separated list that is dealt to the heads in turn (layer, train), or the list of
           patterns (search)
  f32      the raster tensors are float32 (the permutation casts on the way in and out) instead of bfloat16
"""
import math

import torch

import paper_2502_04507_amd as sta

DEVICE = "cuda:0"


def _case(kind, B, H, D, grid, tile, windows, f32=False, name=None):
    case = {"kind": kind, "B": B, "H": H, "D": D, "grid": grid, "tile": tile, "windows": windows, "f32": f32}
    return dict(case, name=name) if name else case


def listed():
    return [
        # A small 3D latent with one head and float32 activations: what unit-sized models and smoke runs call.
        # A few dozen work items: latency and launches.
        _case("layer", 1, 1, 64, "18x24x24", "6x8x8", "1x3x3", f32=True, name="layer_tiny_3d_f32"),
        # One image at inference, 2D tiles of 8x8 tokens, batch 1: interactive latency.
        _case("layer", 1, 8, 64, "1x64x64", "1x8x8", "1x3x3", name="layer_image"),
        # A batch of sixteen such images, the throughput setting of the same model.
        _case("layer", 16, 8, 64, "1x64x64", "1x8x8", "1x3x3", name="layer_image_batch"),
        # A short clip: the middle of the range, a few rounds of work items.
        _case("layer", 1, 12, 128, "12x48x48", "6x8x8", "1x3x3", name="layer_clip"),
        # The full video latent with the window the method is quoted at, same window on every head.
        _case("layer", 1, 24, 128, "30x48x80", "6x8x8", "3x3x3", name="layer_video"),
        # The same layer after a mask search: every head its own window, from local to the whole grid.
        _case("layer", 1, 24, 128, "30x48x80", "6x8x8", "1x3x3,3x3x3,3x3x5,5x6x10", name="layer_video_mixed"),
        # The full video latent for a model of head dimension 64.
        _case("layer", 1, 24, 64, "30x48x80", "6x8x8", "3x3x3", name="layer_video_d64"),
        # A latent whose sides only divide by odd-sized tiles (96 tokens), two prompts, five heads, an even window.
        _case("layer", 2, 5, 128, "10x30x56", "2x6x8", "3x3x3,2x4x3", name="layer_odd_tile"),
        # Finetuning an image model: four images, forward and backward.
        _case("train", 4, 8, 64, "1x64x64", "1x8x8", "1x3x3", name="train_image"),
        # Finetuning on short clips.
        _case("train", 1, 12, 128, "12x48x48", "6x8x8", "1x3x3", name="train_clip"),
        # Finetuning on the full video latent.
        _case("train", 1, 24, 128, "30x48x80", "6x8x8", "3x3x3", name="train_video"),
        # The search that picks every head's window, once per layer and prompt, on the full video latent.
        _case("search", 1, 24, 128, "30x48x80", "6x8x8", "1x3x3,3x3x3,3x3x5", name="search_video"),
    ]


# Tile shapes (multiples of 32 tokens, as the entry points ask for) with how often a drawn case takes them: the video
# tile and the image tile most, the others as they come with latents whose sides divide differently.
_TILES = [((6, 8, 8), 6), ((1, 8, 8), 4), ((2, 8, 8), 3), ((3, 8, 8), 1), ((4, 8, 8), 1), ((2, 6, 8), 1), ((4, 4, 6), 1),
          ((4, 4, 8), 1), ((5, 8, 8), 1), ((1, 4, 8), 1)]
_MOST_FLOPS = {"layer": 4.0e13, "train": 1.5e13, "search": 1.5e13}      # of one pass; an odd tile takes a quarter of it
_LEAST_FLOPS = 5.0e8
_MOST_BYTES = 1.5e9                                                    # of one tensor


def _text(triple):
    return "x".join(str(x) for x in triple)


def _triple(text):
    return tuple(int(x) for x in text.split("x"))


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["train"] * 3 + ["search"])
    aim = _log_uniform(rng, _LEAST_FLOPS, _MOST_FLOPS[kind] / 2)           # sizes spread over the logarithm of the work
    while True:
        tile = rng.choice([t for t, times in _TILES for _ in range(times)])
        P = tile[0] * tile[1] * tile[2]
        D = rng.choice([64, 128])
        n_tiles = _log_uniform(rng, 4, min(600, 131072 / P))
        # sides in tiles: time short, height and width of a similar size
        n_t = 1 if tile[0] == 1 else max(1, min(6, round(n_tiles ** (1 / 3) * rng.uniform(0.4, 1.2))))
        n_h = max(1, round(math.sqrt(n_tiles / n_t) * rng.uniform(0.6, 1.1)))
        n_w = max(1, round(n_tiles / (n_t * n_h)))
        n = (n_t, n_h, n_w)
        H = round(_log_uniform(rng, 1, 40))
        B = rng.choice([1, 1, 1, 2, 3, 4]) if tile[0] > 1 else round(_log_uniform(rng, 1, 24))

        def window():
            return tuple(min(rng.choice([1, 2, 3, 3, 3, 4, 5, 9]), m) for m in n)

        windows = [window()]
        if kind == "search":
            windows, sizes = [], set()          # patterns of different sizes: equal ones would tie on such inputs
            for w in [window() for _ in range(8)]:
                kept = sta.sta_kept_flops(1, 1, D, [a * b for a, b in zip(n, tile)], tile, [w])
                if kept not in sizes and len(windows) < 5:
                    sizes.add(kept)
                    windows.append(w)
            windows = windows[1:]
            if len(windows) < 2:
                continue
        elif rng.random() < 0.4:
            windows = [window() for _ in range(rng.randint(2, 4))] + ([n] if rng.random() < 0.3 else [])
        case = _case(kind, B, H, D, _text([a * b for a, b in zip(n, tile)]), _text(tile), ",".join(_text(w) for w in windows),
                     f32=kind == "layer" and rng.random() < 0.15)
        flops = work(case)["flops"]
        most = _MOST_FLOPS[kind] / (4 if P % 128 else 1)
        if aim / 2 <= flops <= min(2 * aim, most) and 2.0 * B * H * D * P * n_t * n_h * n_w <= _MOST_BYTES:
            return case


def _parse(case):
    grid, tile = _triple(case["grid"]), _triple(case["tile"])
    windows = [_triple(w) for w in case["windows"].split(",")]
    per_head = [windows[h % len(windows)] for h in range(case["H"])]
    return grid, tile, windows, per_head


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.kind = case["kind"]
    s.grid, s.tile, s.patterns, s.windows = _parse(case)
    B, H, D = case["B"], case["H"], case["D"]
    N = s.grid[0] * s.grid[1] * s.grid[2]
    raster = torch.float32 if case["f32"] else torch.bfloat16
    generator = torch.Generator(device=DEVICE)
    generator.manual_seed(seed)

    # activations behind a query/key normalisation: N(0, 1)
    def normal(dtype):
        return torch.randn((B, H, N, D), generator=generator, dtype=torch.float32, device=DEVICE).to(dtype)

    def empty(dtype=torch.bfloat16):
        return torch.empty((B, H, N, D), dtype=dtype, device=DEVICE)

    def scratch(nbytes):
        return torch.empty(max(nbytes, 16), dtype=torch.uint8, device=DEVICE)

    if s.kind == "search":
        s.q_tiled, s.k_tiled, s.v_tiled = (normal(torch.bfloat16) for _ in range(3))
        s.o_full, s.o_pattern = empty(), empty()
        s.workspace = scratch(sta.sta_head_mse_workspace_bytes(B, H))
        s.losses = torch.empty((len(s.patterns), H), dtype=torch.float32, device=DEVICE)
        s.best = torch.empty((H,), dtype=torch.int32, device=DEVICE)
        return s
    s.q, s.k, s.v = (normal(raster) for _ in range(3))
    s.q_tiled, s.k_tiled, s.v_tiled, s.o_tiled = (empty() for _ in range(4))
    s.o = empty(raster)
    if s.kind == "layer":
        s.workspace = scratch(sta.sta_workspace_bytes(B, H, D, s.grid, s.tile))
    else:
        s.d_o = normal(raster)
        s.d_o_tiled = empty()
        s.lse = torch.empty((B, H, N), dtype=torch.float32, device=DEVICE)
        s.d_tiled = [empty() for _ in range(3)]
        s.d = [empty(raster) for _ in range(3)]
        s.workspace = scratch(sta.sta_backward_workspace_bytes(B, H, s.grid))
    return s


def run(s):
    if s.kind == "search":
        sta.sta_mask_search(s.q_tiled, s.k_tiled, s.v_tiled, s.grid, s.tile, s.patterns, s.o_full, s.o_pattern, s.workspace,
                            s.losses, s.best)
        return {"losses": s.losses, "best": s.best}
    sta.sta_tile_permute(s.q, s.q_tiled, s.grid, s.tile)
    sta.sta_tile_permute(s.k, s.k_tiled, s.grid, s.tile)
    sta.sta_tile_permute(s.v, s.v_tiled, s.grid, s.tile)
    if s.kind == "layer":
        sta.sta_forward(s.q_tiled, s.k_tiled, s.v_tiled, s.o_tiled, s.grid, s.tile, s.windows, workspace=s.workspace)
        return sta.sta_untile(s.o_tiled, s.o, s.grid, s.tile)
    sta.sta_forward_lse(s.q_tiled, s.k_tiled, s.v_tiled, s.o_tiled, s.lse, s.grid, s.tile, s.windows)
    sta.sta_untile(s.o_tiled, s.o, s.grid, s.tile)
    sta.sta_tile_permute(s.d_o, s.d_o_tiled, s.grid, s.tile)
    sta.sta_backward(s.q_tiled, s.k_tiled, s.v_tiled, s.o_tiled, s.d_o_tiled, s.lse, *s.d_tiled, s.grid, s.tile, s.windows,
                     s.workspace)
    for tiled, raster in zip(s.d_tiled, s.d):
        sta.sta_untile(tiled, raster, s.grid, s.tile)
    return {"o": s.o, "lse": s.lse, "d_q": s.d[0], "d_k": s.d[1], "d_v": s.d[2]}


def work(case):
    grid, tile, windows, per_head = _parse(case)
    B, H, D = case["B"], case["H"], case["D"]
    N = grid[0] * grid[1] * grid[2]
    tensor = B * H * N * D * (4 if case["f32"] else 2)
    if case["kind"] == "search":
        full = [tuple(g // t for g, t in zip(grid, tile))]
        flops = sum(sta.sta_kept_flops(B, H, D, grid, tile, [w] * H) for w in full + windows)
        return {"bytes": 3 * tensor + 4 * H * (len(windows) + 1), "flops": flops}
    flops = sta.sta_kept_flops(B, H, D, grid, tile, per_head)         # two matrix products over the kept blocks
    if case["kind"] == "layer":
        return {"bytes": 4 * tensor, "flops": flops}
    return {"bytes": 8 * tensor + 4 * B * H * N, "flops": 3.5 * flops}    # five more products in the gradients


def tolerance(case):
    # Probabilities (and dS) are rounded to bfloat16 before the matrix products and the results once more.  Against the
    # same attention in 64 bits that measures 2.1e-3 to 2.9e-3 (2-norm) and up to 0.019 at the worst element, over
    # outputs and gradients of layers and training steps of both head dimensions; about four times that is allowed.
    # "differ" concerns the search's choices only: a head whose two best patterns tie.
    return {"rel": 1e-2, "max": 0.08, "differ": 0.005}
