"""Host only: forwards that read the packed arrays as they are write no part of the workspace, whatever it was sized for, and which kernel computes a forward
does not depend on what the workspace has room for."""
import ctypes

import numpy as np

import paper_2407_11062_amd as eq

TILES, MID, RELAY_MID = 0, 1, 7
WORK, PACKED = 0, 1


def route(T, I, O, bits, g, source):
    out = (ctypes.c_int32 * 3)()
    assert eq.lib().eqat_fwd_route(ctypes.byref(eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)), source, out) == 0
    return out[0]


def parts(T, I, O, bits, g, op, ws_bytes):
    first, end = ctypes.c_size_t(), ctypes.c_size_t()
    d = eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)
    assert eq.lib().eqat_plan_scratch(ctypes.byref(d), op, 0, 256, ws_bytes, ctypes.byref(first), ctypes.byref(end)) == 0
    return end.value - first.value


def test_only_the_tiled_gemm_writes_parts():
    rng = np.random.default_rng(10)
    seen = {TILES: 0, MID: 0, RELAY_MID: 0}
    sizes = [(333, 4096, 11008, 4, 128), (333, 4096, 4096, 4, 256), (100, 11008, 1288, 4, 32), (70, 8192, 1000, 3, 128)]
    for _ in range(3000):
        bits, g = int(rng.integers(2, 5)), int(rng.choice([32, -1]))
        sizes.append((int(np.exp(rng.uniform(0, np.log(4000)))), 32 * int(rng.integers(1, 700)), 8 * int(rng.integers(1, 3000)), bits, g))
    for size in sizes:
        kernel = route(*size, PACKED)
        for op in (eq.OP_Q_FWD, eq.OP_QP_FWD, eq.OP_FQ_FWD, eq.OP_QP_BWD):
            if route(*size, PACKED if op == eq.OP_Q_FWD else WORK) != TILES:
                assert parts(*size, op, 1 << 31) == 0, (size, op)
        seen[kernel] = seen.get(kernel, 0) + 1
    assert min(seen.values()) > 20


def test_sizes_that_one_workgroup_to_a_tile_serves_best_by_the_tiled_gemm():
    # tiles of 64 or 96 tokens shared by several workgroups would be the faster ones by the estimates; unshared they are not
    for size in ((419, 13728, 6848, 2, -1), (1900, 13152, 1880, 4, -1)):
        assert route(*size, PACKED) == route(*size, WORK) == TILES, size
