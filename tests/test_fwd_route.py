"""Which kernel a forward takes, asked on the host (`eqat_fwd_route`, no GPU): the lines of the dispatch rules, and that a
call's kernel does not depend on the entry point from 17 tokens on (the results of all of them are bitwise equal there)."""
import ctypes

import numpy as np
import pytest

import paper_2407_11062_amd as eq

TILES, MID, WIDE, ANY, RUN, SEGMENTS, PAIRS, RELAY_MID = range(8)
WORK, PACKED, FLOATZ = range(3)


def route(T, I, O, bits, g, source=PACKED, act=eq.BF16):
    out = (ctypes.c_int32 * 3)()
    d = eq.make_desc(T, I, O, bits, g, act, eq.BF16)
    rc = eq.lib().eqat_fwd_route(ctypes.byref(d), source, out)
    assert rc == 0, eq.lib().eqat_status_string(rc)
    return tuple(out)


def test_group_sizes_and_token_counts_choose_the_matrix_vector_kernel():
    assert route(1, 4096, 4096, 2, 64)[0] == RUN and route(1, 4096, 4096, 2, -1)[0] == RUN
    assert route(1, 4800, 4096, 2, 96)[0] == ANY and route(1, 1152, 4096, 2, 384)[0] == ANY
    assert route(12, 4096, 4096, 2, 64) == (WIDE, 16, 16) and route(8, 4096, 4096, 2, 64) == (WIDE, 8, 16)
    assert route(4, 28672, 8192, 2, 64)[0] == WIDE                # the token rows exceed the LDS of k_gemv_run
    assert route(17, 4096, 8176, 3, 64) == (WIDE, 32, 16) and route(17, 4096, 8192, 3, 64) == (WIDE, 32, 32)
    assert route(64, 4096, 8176, 3, 64) == (WIDE, 64, 16) and route(64, 8192, 8192, 3, 64) == (WIDE, 64, 32)
    assert route(8192, 4096, 4096, 2, 64) == (TILES, 0, 0)


def test_few_tokens_take_the_faster_of_the_two_matrix_vector_kernels():
    # 3-bit codes, 7 tokens, one group per row: k_gemv_wide; 4-bit codes of many rows, too, but one or two tokens of at most
    # four runs of 1024 inputs with one group per run
    assert route(6, 4096, 11008, 3, -1)[0] == RUN and route(7, 4096, 11008, 3, -1) == (WIDE, 8, 16)
    for g in (256, 512, -1):
        for T in (1, 2):
            assert route(T, 4096, 28672, 4, g)[0] == RUN and route(T, 4608, 28672, 4, 512)[0] == WIDE, (T, g)
        assert route(3, 4096, 28672, 4, g)[0] == WIDE, g
    assert route(1, 4096, 28672, 4, 128)[0] == WIDE and route(1, 8192, 24576, 4, 128)[0] == RUN
    assert route(1, 8192, 24592, 4, 128)[0] == WIDE and route(1, 8192, 28672, 3, 128)[0] == RUN
    # the token rows of up to 16 tokens in the LDS of k_gemv_run: 64 KB at most
    assert route(6, 5440, 4096, 2, 64)[0] == RUN and route(6, 5504, 4096, 2, 64)[0] == WIDE


def test_large_matrices_go_segment_by_segment_where_that_is_faster():
    large, small = (4096, 8208), (4096, 8192)                     # just above and at 2^25 weights
    for bits, g, source in ((2, 64, PACKED), (2, 64, FLOATZ), (2, 32, FLOATZ), (3, 32, FLOATZ), (3, 128, FLOATZ), (4, 32, FLOATZ), (4, 64, FLOATZ)):
        assert route(1, *large, bits, g, source)[0] == SEGMENTS and route(1, *small, bits, g, source)[0] == RUN, (bits, g, source)
    for bits, g, source in ((2, 32, PACKED), (2, 128, FLOATZ), (3, 64, PACKED), (3, 256, FLOATZ), (4, 64, PACKED), (4, 128, FLOATZ)):
        assert route(1, *large, bits, g, source)[0] == RUN, (bits, g, source)
    assert route(2, *large, 2, 64)[0] == SEGMENTS and route(3, *large, 2, 64)[0] == RUN
    assert route(2, 2048, 24584, 2, 64)[0] == PAIRS and route(2, 2048, 24576, 2, 64)[0] == SEGMENTS
    assert route(2, 2112, 24584, 2, 64)[0] == SEGMENTS and route(3, 1344, 60000, 2, 64)[0] == PAIRS
    assert route(1, 512, 60000, 2, 64)[0] == PAIRS and route(4, 1024, 60000, 2, 64)[0] == RUN
    assert route(4, 1024, 32768, 2, 64)[0] == PAIRS and route(4, 1024, 32776, 2, 64)[0] == RUN
    for source in (PACKED, FLOATZ):                               # 6144 and 6160 waves of k_gemv_run
        assert route(1, 4096, 24576, 2, 64, source)[0] == SEGMENTS and route(1, 4096, 24584, 2, 64, source)[0] == PAIRS
        assert route(2, 4096, 28672, 2, 64, source)[0] == SEGMENTS and route(1, 4096, 28672, 2, 128, source)[0] == RUN
    assert route(6, *large, 3, 64, FLOATZ)[0] == SEGMENTS and route(7, *large, 3, 64, FLOATZ)[0] == WIDE


def test_3_bit_codes_are_relaid_where_two_rounds_rebuild_them():
    for T, I, O in ((1300, 11008, 4096), (384, 8192, 11008), (450, 3520, 8200)):
        assert route(T, I, O, 3, 32) == route(T, I, O, 3, 32, FLOATZ) == (RELAY_MID, 96, 128), (T, I, O)
        assert route(T, I, O, 2, 32) == route(T, I, O, 4, 32) == route(T, I, O, 3, 32, WORK) == (MID, 96, 128)
    assert route(333, 4096, 4096, 3, 128)[0] == MID and route(192, 4096, 28672, 3, 128) == (MID, 96, 128)


def test_one_round_of_short_token_tiles_takes_the_kernel_for_few_tiles():
    # from 641 inputs on, whatever the estimates of both kernels say (they overrate this one where the contraction is short)
    for T, I, O, bits, g in ((443, 832, 552, 2, 32), (85, 800, 2504, 3, 32), (135, 800, 2120, 4, 32), (825, 896, 552, 2, 128), (174, 1184, 2792, 3, 32),
                             (101, 864, 3528, 4, -1), (725, 672, 632, 4, -1)):
        assert route(T, I, O, bits, g) == (MID, 64, 128) and route(T, I, O, bits, g, WORK) == (MID, 64, 128), (T, I, O)
    assert route(1389, 896, 1936, 3, 128) == (MID, 96, 128)
    assert route(443, 640, 552, 2, 32)[0] == TILES and route(2026, 704, 1672, 2, -1)[0] == TILES          # 640 inputs; two rounds


def test_the_entry_point_does_not_matter_from_17_tokens_on():
    rng = np.random.default_rng(7)
    seen = set()
    for _ in range(3000):
        T, I, O = int(np.exp(rng.uniform(np.log(17), np.log(3000)))), 32 * int(rng.integers(1, 400)), 8 * int(rng.integers(1, 3000))
        g = int(rng.choice([32, I]))
        bits = int(rng.integers(2, 5))
        a, b, c = (route(T, I, O, bits, g, source) for source in (WORK, PACKED, FLOATZ))
        assert b == c and a[1:] == b[1:] and a[0] == (MID if b[0] == RELAY_MID else b[0]), (T, I, O, bits, g, a, b, c)
        seen.add(a[:2])
    assert seen >= {(WIDE, 32), (WIDE, 64), (MID, 64), (MID, 96), (TILES, 0)}
    for T in range(1, 17):                                        # fewer: only the packed arrays have a kernel of their own
        assert route(T, 4096, 4096, 2, 64, WORK)[0] == TILES


def test_bad_arguments():
    L = eq.lib()
    out = (ctypes.c_int32 * 3)()
    ok = eq.make_desc(4, 512, 512, 2, 32, eq.BF16, eq.BF16)
    assert L.eqat_fwd_route(ctypes.byref(ok), 1, out) == 0
    assert L.eqat_fwd_route(ctypes.byref(ok), 1, None) != 0 and L.eqat_fwd_route(None, 1, out) != 0
    for bad in (eq.make_desc(0, 512, 512, 2, 32, eq.BF16, eq.BF16), eq.make_desc(4, 512, 512, 2, 32, eq.F32, eq.F32),
                eq.make_desc(4, 512, 512, 5, 32, eq.BF16, eq.BF16), eq.make_desc(4, 500, 512, 2, 32, eq.BF16, eq.BF16)):
        assert L.eqat_fwd_route(ctypes.byref(bad), 1, out) != 0
