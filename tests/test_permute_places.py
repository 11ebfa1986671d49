"""Where the permutation kernels read and write, evaluated on the host by the functions that the kernels call: every piece of small
tensors, and pieces of tensors whose planes hold 2^32 and more chunks of 8 elements (64 GB, of which no memory is needed here)."""
import ctypes

import numpy as np
import pytest

import paper_2502_04507_amd as sta

BF16, F32 = 0, 1
NONE = 2 ** 64 - 1
I3 = ctypes.c_int * 3


def piece_of(types, B, H, D, grid, tile, workgroup, piece):
    raster, tiled = ctypes.c_uint64(), ctypes.c_uint64()
    status = sta.load_library().sta_permuted_piece(*types, B, H, D, I3(*grid), I3(*tile), ctypes.c_uint32(workgroup), ctypes.c_uint32(piece),
                                                   ctypes.byref(raster), ctypes.byref(tiled))
    assert status == 0, sta.sta_strerror(status)
    return raster.value, tiled.value


def raster_of(tiled, D, grid, tile):
    """The raster chunk of a tiled chunk, in Python's integers."""
    token, chunk = divmod(tiled, D // 8)
    n = [g // t for g, t in zip(grid, tile)]
    slice_and_tile, inside = divmod(token, tile[0] * tile[1] * tile[2])
    outer, tile_id = divmod(slice_and_tile, n[0] * n[1] * n[2])
    at = []
    for ext, m in zip(reversed(tile), reversed(n)):
        inside, i = divmod(inside, ext)
        tile_id, j = divmod(tile_id, m)
        at.append(j * ext + i)
    w, h, t = at
    return (((outer * grid[0] + t) * grid[1] + h) * grid[2] + w) * (D // 8) + chunk


@pytest.mark.parametrize("types,lanes", [((BF16, BF16), 256), ((F32, BF16), 512)])
@pytest.mark.parametrize("slices,D,grid,tile", [
    (2, 8, (4, 16, 33), (1, 1, 1)), (3, 64, (1, 24, 24), (1, 4, 8)), (5, 72, (3, 10, 14), (3, 5, 7)), (7, 64, (2, 9, 12), (2, 3, 12)),
], ids=str)
def test_every_chunk_is_moved_once_and_to_its_place(slices, D, grid, tile, types, lanes):
    per_tile = tile[0] * tile[1] * tile[2] * D // 8
    chunks = slices * grid[0] * grid[1] * grid[2] * D // 8
    workgroups = chunks // per_tile * -(-per_tile // lanes)
    seen = []
    for workgroup in range(workgroups):
        for piece in range(lanes):
            raster, tiled = piece_of(types, 1, slices, D, grid, tile, workgroup, piece)
            if tiled != NONE:
                assert raster == raster_of(tiled, D, grid, tile), (workgroup, piece)
                seen.append(tiled)
    assert sorted(seen) == list(range(chunks))
    assert piece_of(types, 1, slices, D, grid, tile, workgroups, 0) == (NONE, NONE)


@pytest.mark.parametrize("slices,D,grid,tile", [
    (2, 128, (1, 16384, 16384), (1, 8, 8)),         # a plane of 2^32 chunks; the second slice stands behind it
    (2, 64, (1, 32768, 16384), (1, 8, 8)),
    (1, 64, (2, 32768, 16384), (1, 8, 8)),          # and the second layer of tiles
    (1, 128, (2, 16384, 16384), (2, 8, 8)),         # the second plane of a tile
    (2, 128, (1, 512, 1920000), (1, 512, 64)),      # runs of one tile 2^32 chunks and more apart, in the same plane
    (1, 1024, (1, 1024, 65536), (1, 512, 8)),       # from a tile to the next along h
    (3, 128, (3, 10240, 16384), (3, 8, 8)),         # 0.6 of that a plane
], ids=str)
def test_places_in_tensors_of_64_gb_and_more(slices, D, grid, tile):
    per_tile = tile[0] * tile[1] * tile[2] * D // 8
    parts = -(-per_tile // 256)
    workgroups = slices * grid[0] * grid[1] * grid[2] * D // 8 // per_tile * parts
    rng = np.random.default_rng(5)
    ids = {0, workgroups - 1} | set(int(x) for x in rng.integers(0, workgroups, 3000))
    seen = set()
    for workgroup in ids:
        piece = int(rng.integers(0, min(per_tile, 256)))
        raster, tiled = piece_of((BF16, BF16), 1, slices, D, grid, tile, workgroup, piece)
        if tiled == NONE:
            continue
        assert raster == raster_of(tiled, D, grid, tile), (workgroup, piece)
        seen.add(raster)
    assert len(seen) > 2900 and max(seen) > 2 ** 32
