"""Where launches put the accumulator parts of tiles that several workgroups share: inside the workspace that the call was given, on a GPU of
any number of compute units (host only: `eqat_plan_scratch` asks the functions that plan the launches)."""
import ctypes

import numpy as np
import pytest

import paper_2407_11062_amd as eq

OPS = {eq.OP_FQ_FWD: 1, eq.OP_FQ_BWD: 3, eq.OP_Q_FWD: 1, eq.OP_Q_BWD: 3, eq.OP_QP_FWD: 1, eq.OP_QP_BWD: 3}      # GEMMs that a call launches


def need(T, I, O, op, bits=2, g=32):
    return eq.lib().eqat_workspace_bytes(ctypes.byref(eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)), op)


def parts(T, I, O, op, gemm, cus, ws_bytes, bits=2, g=32):
    """(first, past the last) byte of the workspace that the launch writes parts to; None: the call refuses that workspace"""
    first, end = ctypes.c_size_t(), ctypes.c_size_t()
    d = eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)
    rc = eq.lib().eqat_plan_scratch(ctypes.byref(d), op, gemm, cus, ws_bytes, ctypes.byref(first), ctypes.byref(end))
    assert rc in (0, 7), eq.lib().eqat_status_string(rc)
    return None if rc else (first.value, end.value)


def ragged_shapes(n, seed):
    rng = np.random.default_rng(seed)
    for _ in range(n):
        T = int(np.exp(rng.uniform(0, np.log(9000))))
        I = 32 * int(np.exp(rng.uniform(np.log(4), np.log(700))))
        yield T, I, 8 * int(np.exp(rng.uniform(np.log(16), np.log(3000))))


@pytest.mark.parametrize("cus", [256, 208, 128, 64, 32, 8])
def test_parts_stay_inside_the_workspace_on_any_number_of_compute_units(cus):
    written = set()
    # 4096 tokens, 512 -> 20480: 256 compute units share the tiles of dX alone, 128 would cut those of dW, whose parts are larger
    for T, I, O in [(4096, 512, 20480), (1280, 4096, 4096), (2560, 2048, 5504), (8192, 4096, 11008), *ragged_shapes(4000, 5)]:
        for op in (eq.OP_FQ_BWD, eq.OP_Q_FWD, eq.OP_QP_BWD):
            ws_bytes = need(T, I, O, op)
            for gemm in range(OPS[op]):
                first, end = parts(T, I, O, op, gemm, cus, ws_bytes)
                assert end <= ws_bytes, (T, I, O, op, gemm, first, end, ws_bytes)
                if end > first:
                    written.add(gemm)
    assert written == {0, 1, 2} or cus < 256


@pytest.mark.parametrize("I,O", [(4096, 4096), (11008, 4096), (8192, 1024)])
def test_a_workspace_sized_for_many_tokens_serves_few(I, O):
    for op, gemms in OPS.items():
        ws_bytes = need(8192, I, O, op)
        for T in (1, 2, 17, 64, 128, 256, 333, 515, 1000, 1280, 2048):
            for gemm in range(gemms):
                first, end = parts(T, I, O, op, gemm, 256, ws_bytes)          # not refused
                assert end <= ws_bytes


def test_what_the_codes_and_pairs_take_is_still_asked_for():
    for op in OPS:
        first, _ = parts(256, 4096, 4096, op, 0, 256, 1 << 30)
        assert parts(256, 4096, 4096, op, 0, 256, first) == (first, first)     # no room for parts: none are written
        assert parts(256, 4096, 4096, op, 0, 256, first - 1) is None
    # tiles that are cut because they do not fill whole rounds need their parts, as ever: 13B q projection, 320 tiles
    for op in (eq.OP_Q_FWD, eq.OP_QP_BWD):
        n = need(4096, 5120, 5120, op)
        assert parts(4096, 5120, 5120, op, 0, 256, n)[1] <= n and parts(4096, 5120, 5120, op, 0, 256, n - 256) is None


def test_more_workspace_than_asked_for_changes_no_plan():
    for T, I, O in ragged_shapes(500, 6):
        for cus in (256, 128):
            n = need(T, I, O, eq.OP_FQ_BWD)
            for gemm in range(3):
                assert parts(T, I, O, eq.OP_FQ_BWD, gemm, cus, n) == parts(T, I, O, eq.OP_FQ_BWD, gemm, cus, n + (1 << 28))


def test_no_room_for_parts_that_no_launch_writes():
    """Whatever the kernel of the forward: the workspace ends where the last launch that writes parts ends, or where they would begin."""
    seen = set()
    for T, I, O in [(1, 4096, 4096), (1, 4096, 11008), (8, 5120, 13824), (333, 4096, 4096), (333, 4096, 11008), *ragged_shapes(3000, 7)]:
        for op in (eq.OP_Q_FWD, eq.OP_QP_FWD, eq.OP_FQ_FWD):
            n = need(T, I, O, op)
            first, end = parts(T, I, O, op, 0, 256, n)
            assert n == end, (T, I, O, op, first, end, n)
            seen.add((op, end > first))
    assert len(seen) == 6
    # decoding: codes of the working layout, pairs, counters and no more
    assert need(1, 4096, 4096, eq.OP_Q_FWD, 2, 64) == 4096 * 4096 // 4 + 4096 * 64 * 8 + 8192


def test_split_tiles_have_one_part_per_workgroup():
    """Runs begin and end inside tiles: two parts per workgroup.  A split or shared tile takes one of each of its workgroups."""
    part = 256 * 256 * 4
    for shape, gemm, slots in (((1280, 4096, 4096), 1, 1), ((4096, 5120, 5120), 0, 1), ((4096, 5120, 6656), 0, 2)):
        first, end = parts(*shape, eq.OP_FQ_BWD, gemm, 256, 1 << 30)
        assert end - first == 256 * slots * part, shape
