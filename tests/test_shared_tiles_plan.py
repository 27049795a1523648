"""How k_gemm_ksplit divides a forward or dX with few output tiles among workgroups (host only: `eqat_shared_item` calls the function that
tells a workgroup its share): every K-tile pair of every tile exactly once, parts in order and of equal length but for one pair."""
import ctypes

import numpy as np
import pytest

import paper_2407_11062_amd as eq
from test_fwd_route import TILES, WORK, route


def dx_tokens(T, I, O, bits=2, g=32):
    route = (ctypes.c_int32 * 2)()
    assert eq.lib().eqat_dx_route(ctypes.byref(eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)), 1, route) == 0
    return route[0]


def shared_items(T, I, O, gemm, bits=2, g=32):
    """items of all workgroups; none where another kernel computes this GEMM"""
    d = eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)
    item, exists, out = (ctypes.c_int32 * 10)(), ctypes.c_int32(), []
    while True:
        assert eq.lib().eqat_shared_item(ctypes.byref(d), gemm, len(out), item, ctypes.byref(exists)) == 0
        if not exists.value:
            return out
        out.append(tuple(item))


def parts_of(T, I, O, gemm, bits=2, g=32):
    items = shared_items(T, I, O, gemm, bits, g)
    return items[0][5] if items else 0


def check(T, I, O, gemm):
    items = shared_items(T, I, O, gemm)
    if not items:
        return 0
    M, N, K = (T, O, I) if gemm == 0 else (T, I, O)
    parts, grid, pairs, tiles_m, tiles_n = items[0][5:]
    assert (tiles_m, tiles_n, pairs) == (-(-M // 128), -(-N // 128), -(-K // 128))
    assert 1 <= parts <= 4 and len(items) == grid == tiles_m * tiles_n * parts <= 256 and pairs >= (4 * parts if parts > 1 else 1)
    cover = np.zeros((tiles_m, tiles_n, pairs), np.int32)
    where = {}
    for tm, tn, kb, ke, part, *rest in items:
        assert tuple(rest) == (parts, grid, pairs, tiles_m, tiles_n)
        assert 0 <= tm < tiles_m and 0 <= tn < tiles_n and 0 <= kb < ke <= pairs
        cover[tm, tn, kb:ke] += 1
        where[tm, tn, part] = (kb, ke)
    assert (cover == 1).all() and len(where) == grid
    for tm in range(tiles_m):
        for tn in range(tiles_n):
            ranges = [where[tm, tn, k] for k in range(parts)]
            assert all(a[1] == b[0] for a, b in zip(ranges, ranges[1:]))                # in the order in which they are added up
            sizes = [ke - kb for kb, ke in ranges]
            assert max(sizes) - min(sizes) <= 1
    return parts


def test_every_pair_of_every_tile_is_computed_once():
    rng = np.random.default_rng(11)
    seen = set()
    for _ in range(500):
        T = int(np.exp(rng.uniform(0, np.log(4000))))
        I = 32 * int(np.exp(rng.uniform(0, np.log(900))))
        O = 8 * int(np.exp(rng.uniform(0, np.log(3600))))
        for gemm in (0, 1):
            seen.add((gemm, check(T, I, O, gemm)))
    assert seen >= {(1, k) for k in range(5)} | {(0, 0), (0, 1), (0, 4)}


def test_known_launches():
    assert parts_of(256, 4096, 11008, 1) == 4 and parts_of(1000, 4096, 2048, 1) == 1           # dX: 64 tiles, 256 tiles
    assert parts_of(256, 11008, 4096, 1) == 1 and parts_of(1280, 4096, 4096, 1) == 0           # 172 tiles; 320: the tile kernels
    assert parts_of(1, 4096, 4096, 0) == 4 and route(1, 4096, 4096, 2, 32, WORK)[0] == TILES   # one token on a prepared layer
    assert parts_of(333, 4096, 4096, 0) == 0                                                   # k_gemm_mid
    # two or four whole K tiles: the tile kernel; any other length up to them is shared by the two K groups
    for K, parts in ((32, 1), (64, 1), (96, 1), (128, 0), (160, 1), (192, 1), (256, 0), (288, 1), (384, 1)):
        assert parts_of(100, K, 512, 0) == parts and parts_of(1000, 4096, K, 1) == parts, K


def test_none_where_the_kernel_for_few_tiles_computes_dx():
    """256 tiles of 128 x 128 and a long contraction, a handful of tiles and a short one: k_gemm_mid_dx (`eqat_dx_route`) and no other."""
    for T, I, O in ((1000, 4096, 4096), (100, 512, 96), (70, 96, 40), (300, 352, 200)):
        assert dx_tokens(T, I, O) != 0 and shared_items(T, I, O, 1) == [] and parts_of(T, I, O, 1) == 0
    rng = np.random.default_rng(12)
    seen = set()
    for _ in range(500):
        T, I, O = int(np.exp(rng.uniform(0, 8))), 32 * int(np.exp(rng.uniform(0, 6))), 8 * int(np.exp(rng.uniform(0, 8)))
        way = (dx_tokens(T, I, O) != 0, bool(shared_items(T, I, O, 1)))
        assert way != (True, True), (T, I, O)
        seen.add(way)
    assert len(seen) == 3


def test_bad_arguments():
    L, item, ex = eq.lib(), (ctypes.c_int32 * 10)(), ctypes.c_int32()
    r = ctypes.byref(eq.make_desc(512, 512, 512, 2, 32, eq.BF16, eq.BF16))
    assert L.eqat_shared_item(r, 0, 0, item, ctypes.byref(ex)) == 0 and ex.value == 1
    assert L.eqat_shared_item(r, 0, 1 << 20, item, ctypes.byref(ex)) == 0 and ex.value == 0
    for bad in ((2, 0), (-1, 0), (0, -1)):
        assert L.eqat_shared_item(r, *bad, item, ctypes.byref(ex)) != 0
    assert L.eqat_shared_item(r, 0, 0, None, ctypes.byref(ex)) != 0 and L.eqat_shared_item(r, 0, 0, item, None) != 0
    f32 = eq.make_desc(512, 512, 512, 2, 32, eq.F32, eq.F32)
    assert L.eqat_shared_item(ctypes.byref(f32), 0, 0, item, ctypes.byref(ex)) != 0
